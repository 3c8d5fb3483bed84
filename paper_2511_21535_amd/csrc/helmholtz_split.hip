// Near-field Helmholtz in single precision on the BF16 matrix cores, without
// giving up single precision: every FP32 operand is the exact sum of three
// BF16 values, x = h + m + l (8 significand bits each, the exponent range of
// FP32), and a real product takes the six partial products of order up to two,
// h h, h m, m h, m m, h l, l h, accumulated in FP32 by
// v_mfma_f32_32x32x16_bf16.  What is left out (m l, l m, l l) lies below
// 2^-23 of the product, as one FP32 rounding does, while the sixteen terms an
// instruction adds are rounded once instead of eight times: the error against
// 64 bits of a 64^3 grid is 1.4e-7 where FP32 matrix instructions (three real
// products per complex one) leave 2.2e-7.  A BF16 product takes a sixteenth of
// the FP32 one's time, so six cost 0.38 of it.  The parts do not hold
// what lies below 2^-133 (q of 1e-36 would be off by 1e-3), a value that rounds
// to infinity in BF16, nor infinities.  A wavefront whose sums tell of one
// forms them again on the FP32 matrix cores.
#include <algorithm>
#include <type_traits>

#include "helm_columns.h"

namespace p2p {
namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float floatx16 __attribute__((ext_vector_type(16)));
typedef float floatx4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

// The packed conversion as one instruction: from plain casts the compiler
// converts the low value a second time wherever it is also used as a float.
__device__ inline uint32_t bf16_pair(float a, float b) {
    uint32_t r;
    asm("v_cvt_pk_bf16_f32 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b));
    return r;
}
__device__ inline float bf16_lo(uint32_t v) { return __uint_as_float(v << 16); }
__device__ inline float bf16_hi(uint32_t v) { return __uint_as_float(v & 0xffff0000u); }

// Two values into their three BF16 parts, packed in pairs.  Each difference is
// exact: what is left after rounding to 8 bits fits in the remaining 16.
__device__ inline void split_rest(float a, float b, uint32_t h, uint32_t &m, uint32_t &l) {
    const float a1 = a - bf16_lo(h), b1 = b - bf16_hi(h);
    m = bf16_pair(a1, b1);
    l = bf16_pair(a1 - bf16_lo(m), b1 - bf16_hi(m));
}
__device__ inline void split_pair(float a, float b, uint32_t &h, uint32_t &m, uint32_t &l) {
    h = bf16_pair(a, b);
    split_rest(a, b, h, m, l);
}
// The same, the bits of both values added to nz.  In one block with the
// conversion: by itself the compiler puts the addition off and keeps the values in
// their registers until then (20 more, with spills).
__device__ inline void split_pair(float a, float b, uint32_t &h, uint32_t &m, uint32_t &l, uint32_t &nz) {
    asm("v_cvt_pk_bf16_f32 %0, %2, %3\n\tv_or3_b32 %1, %1, %2, %3" : "=&v"(h), "+v"(nz) : "v"(a), "v"(b));
    split_rest(a, b, h, m, l);
}
// Im G = sin(kh r) / (4 pi r) below what the parts hold, at every distance
__device__ inline bool unheld_kh(double kh) { return kh > 0.0 && kh < 0x1p-98; }

// A wavefront's sums again on the FP32 matrix cores, which hold every FP32 value
// and keep an infinite source to the targets that it reaches: over the offsets in
// `offs`, G from its 148 values (formed here, s_g may be shared by the wavefronts
// of one table), four real products per complex one, 32 sources at a time added
// in double.  row[o * cap] is the first source row of this lane's column at offset
// o; conj: the sums of conj(q), as in the products.  Functions of their own, so
// that their registers do not count in the products.  With every wavefront taken
// again (q of 1e-36) a prepared 64^3 call takes 79 us instead of 33, one of 20
// right-hand sides on 44^3 448 us instead of 147.
struct RedoSource {
    const int64_t *row;
    int cap;
    const float2 *src, *zeros;
    int32_t nrhs, rhs;
    bool conj;
    // rows of offset o: the first entry and the stride
    __device__ const float2 *open(int o, int64_t &stride) const {
        const int64_t first = row[o * cap];
        stride = first >= 0 ? nrhs : 1;
        return first >= 0 ? src + first * nrhs + rhs : zeros;
    }
};
__device__ inline void green_values(double kh, float2 *s_g) {
    for (int dd = threadIdx.x & 63; dd < kDistances; dd += 64) {
        const double2 v = green(kh, dd);
        s_g[dd] = make_float2(static_cast<float>(v.x), static_cast<float>(v.y));
    }
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
    __builtin_amdgcn_wave_barrier();
}
// 32 columns, the targets 32 rt + 0..31: out[16][2][64] as k_helm_split_cols holds them.
template <class S>
__device__ __attribute__((noinline)) void redo_half_tile(uint32_t offs, double kh, float2 *s_g, RedoSource f, int rt,
                                                         S *out) {
    const int lane = threadIdx.x & 63, i = 32 * rt + (lane & 31), half = lane >> 5;
    green_values(kh, s_g);
    double sr[16], si[16];
#pragma unroll
    for (int r = 0; r < 16; ++r) sr[r] = si[r] = 0.0;
    for (; offs != 0; offs &= offs - 1) {
        const int o = __ffs(offs) - 1;
        int64_t stride;
        const float2 *q = f.open(o, stride) + half * stride;
#pragma unroll 1
        for (int s0 = 0; s0 < 64; s0 += 32) {
            floatx16 re = floatx16{0}, im = floatx16{0};
#pragma unroll 4
            for (int s = s0 + half; s < s0 + 32; s += 2, q += 2 * stride) {
                const float x = q->x, y = f.conj ? -q->y : q->y;
                const float2 g = s_g[near_distance(o, s, i)];
                re = __builtin_amdgcn_mfma_f32_32x32x2f32(g.x, x, re, 0, 0, 0);
                im = __builtin_amdgcn_mfma_f32_32x32x2f32(g.x, y, im, 0, 0, 0);
                re = __builtin_amdgcn_mfma_f32_32x32x2f32(g.y, -y, re, 0, 0, 0);
                im = __builtin_amdgcn_mfma_f32_32x32x2f32(g.y, x, im, 0, 0, 0);
            }
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                sr[r] += static_cast<double>(re[r]);
                si[r] += static_cast<double>(im[r]);
            }
        }
    }
#pragma unroll
    for (int r = 0; r < 16; ++r) {
        out[(2 * r) * 64 + lane] = static_cast<S>(sr[r]);
        out[(2 * r + 1) * 64 + lane] = static_cast<S>(si[r]);
    }
}
// 16 columns, all 64 targets, stored (if this lane's column is one) to the
// caller's rows row_of[target] of u, times sc.
__device__ __attribute__((noinline)) void redo_columns(uint32_t offs, double kh, float2 *s_g, RedoSource f, bool mine,
                                                       const int32_t *row_of, float sc, float2 *u) {
    const int lane = threadIdx.x & 63, col = lane & 15, kq = lane >> 4;
    green_values(kh, s_g);
    double sr[16], si[16];
#pragma unroll
    for (int r = 0; r < 16; ++r) sr[r] = si[r] = 0.0;
    for (; offs != 0; offs &= offs - 1) {
        const int o = __ffs(offs) - 1;
        int64_t stride;
        const float2 *q = f.open(o, stride) + kq * stride;
#pragma unroll 1
        for (int s0 = 0; s0 < 64; s0 += 32) {
            floatx4 re[4], im[4];
#pragma unroll
            for (int rt = 0; rt < 4; ++rt) re[rt] = im[rt] = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll 2
            for (int s = s0 + kq; s < s0 + 32; s += 4, q += 4 * stride) {
                const float x = q->x, y = f.conj ? -q->y : q->y;
#pragma unroll
                for (int rt = 0; rt < 4; ++rt) {
                    const float2 g = s_g[near_distance(o, s, 16 * rt + col)];
                    re[rt] = __builtin_amdgcn_mfma_f32_16x16x4f32(g.x, x, re[rt], 0, 0, 0);
                    im[rt] = __builtin_amdgcn_mfma_f32_16x16x4f32(g.x, y, im[rt], 0, 0, 0);
                    re[rt] = __builtin_amdgcn_mfma_f32_16x16x4f32(g.y, -y, re[rt], 0, 0, 0);
                    im[rt] = __builtin_amdgcn_mfma_f32_16x16x4f32(g.y, x, im[rt], 0, 0, 0);
                }
            }
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                sr[r] += static_cast<double>(re[r / 4][r % 4]);
                si[r] += static_cast<double>(im[r / 4][r % 4]);
            }
        }
    }
    if (!mine) return;
#pragma unroll
    for (int r = 0; r < 16; ++r) {
        const float x = static_cast<float>(sr[r] * sc), y = static_cast<float>(si[r] * sc);
        u[static_cast<int64_t>(row_of[16 * (r / 4) + 4 * kq + r % 4]) * f.nrhs + f.rhs] = make_float2(x, f.conj ? -y : y);
    }
}

// Whether a wavefront's sums tell of values that the parts do not hold.  What lies
// below 2^-133, the subnormal spacing of BF16, is lost, and a value that rounds to
// infinity in BF16 leaves NaN; so a sum of at most 1728 products with |G| < 0.08 is
// off by less than 2^-127, or NaN.  Sums of 2^-100 and more are good; smaller ones,
// and columns of which every sum is zero, are not, unless they are sums of
// nothing: nz_r and nz_i hold the bits of every Re q and Im q (a column's values
// and sums lie in the 64 / C lanes l, l + C, ... that hold it; with kh = 0 the
// parts do not mix).  A single zero is good: a target may be the only source, or
// its terms cancel.
struct SumBits {
    uint32_t least = ~0u, most = 0;   // the least nonzero (less one) and the greatest of the magnitudes
    __device__ void add(float x) {
        const uint32_t b = __float_as_uint(x) & 0x7fffffffu;
        least = min(least, b - 1u);
        most = max(most, b);
    }
};
template <int C, int NR, class S>
__device__ inline bool sums_unheld(double kh, uint32_t nz_r, uint32_t nz_i, const S (&sr)[NR], const S (&si)[NR]) {
    SumBits r, i;
#pragma unroll
    for (int k = 0; k < NR; ++k) {
        r.add(static_cast<float>(sr[k]));
        i.add(static_cast<float>(si[k]));
    }
#pragma unroll
    for (int d = C; d < 64; d <<= 1) {
        nz_r |= __shfl_xor(nz_r, d, 64);
        nz_i |= __shfl_xor(nz_i, d, 64);
        r.most = max(r.most, static_cast<uint32_t>(__shfl_xor(r.most, d, 64)));
        i.most = max(i.most, static_cast<uint32_t>(__shfl_xor(i.most, d, 64)));
    }
    const uint32_t mix = kh != 0.0 ? ~0u : 0u;
    auto bad = [&](const SumBits &b, uint32_t nz) {
        const bool small = b.most == 0 || b.least < ((127u - 100u) << 23) - 1u;
        return (nz << 1) != 0 && (small || b.most >= (255u << 23));
    };
    return __ballot(bad(r, nz_r | (nz_i & mix)) || bad(i, nz_i | (nz_r & mix))) != 0 || unheld_kh(kh);
}

// G operands of the split products: for table t, copy c, box offset o and run
// s8 of eight sources (8 s8 + 0..7), six planes -- the h, m and l parts of Re G
// and of Im G, each formed in double and rounded to single once -- of 64
// targets x 16 bytes: the operand of a lane of either instruction shape, which
// differ only in which runs and targets their lanes take.  Behind them 63 +
// nrhs zero entries, the sources of an absent neighbour (64 rows from a
// column's right-hand side on, stride one).  G depends on the squared distance
// alone, so a workgroup forms the 148 values it can take once, in double.  The
// workgroups past the first g_wgs (all of them with a prepared plan) copy q into
// sorted order: one launch for what a product needs beforehand.
constexpr int kSplitTable = 27 * 8 * 6 * 64;     // 16-byte operands of a table
constexpr int kSplitTableWgs = 27 * 8 * 64 / 256;
__global__ __launch_bounds__(256) void k_split_prep(const double *__restrict__ kh_dev, HelmInline inl,
                                                    int32_t n_tables, int32_t copies, int32_t nrhs,
                                                    u32x4 *__restrict__ out, int32_t g_wgs,
                                                    const float2 *__restrict__ q, const int32_t *__restrict__ perm,
                                                    uint32_t units, float2 *__restrict__ sorted) {
    __shared__ float2 s_g[kDistances];
    const int tid = threadIdx.x;
    if (static_cast<int32_t>(blockIdx.x) >= g_wgs) {
        permute_entries(q, perm, units, static_cast<uint32_t>(nrhs), sorted, blockIdx.x - static_cast<uint32_t>(g_wgs));
        return;
    }
    constexpr int wgs = kSplitTableWgs;
    const int tab = static_cast<int>(blockIdx.x) / wgs;
    if (tid < kDistances) {
        const double2 v = green(table_kh(inl, kh_dev, tab), tid);
        s_g[tid] = make_float2(static_cast<float>(v.x), static_cast<float>(v.y));
    }
    __syncthreads();
    const int t = (static_cast<int>(blockIdx.x) % wgs) * 256 + tid;
    const int i = t & 63, s8 = (t >> 6) & 7, o = t >> 9;
    u32x4 v[6];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const float2 a = s_g[near_distance(o, 8 * s8 + 2 * j, i)], b = s_g[near_distance(o, 8 * s8 + 2 * j + 1, i)];
        uint32_t h, m, l;
        split_pair(a.x, b.x, h, m, l);
        v[0][j] = h;
        v[1][j] = m;
        v[2][j] = l;
        split_pair(a.y, b.y, h, m, l);
        v[3][j] = h;
        v[4][j] = m;
        v[5][j] = l;
    }
    for (int c = 0; c < copies; ++c) {
        u32x4 *w = out + (static_cast<int64_t>(tab) * copies + c) * kSplitTable + (o * 8 + s8) * 6 * 64 + i;
#pragma unroll
        for (int p = 0; p < 6; ++p) w[p * 64] = v[p];
    }
    float2 *z = reinterpret_cast<float2 *>(out + static_cast<int64_t>(n_tables) * copies * kSplitTable);
    for (int64_t k = static_cast<int64_t>(blockIdx.x) * 256 + tid; k < 63 + static_cast<int64_t>(nrhs);
         k += static_cast<int64_t>(g_wgs) * 256)
        z[k] = make_float2(0.f, 0.f);
}

// (target box, right-hand side) columns, 32 to a tile.  Two workgroups of eight
// wavefronts share a tile, each taking 32 of the 64 targets: a G block's half
// then serves 32 columns, which keeps the operands a workgroup reads from L2
// (0.66 MB of G, 0.2-0.4 MB of Q) below what the matrix cores take to consume
// them.  The wavefronts split the offsets that occur in the tile (wave w the
// w-th, (w + 8)-th, ... of them) and add their partial products in LDS, so a
// workgroup with its CU to itself runs two wavefronts per SIMD, one splitting
// its Q values on the vector unit while the other multiplies.  Four real
// products per complex one: three would save a quarter of the matrix
// instructions but need a third set of G planes, and L2 bounds the kernel as
// much as the matrix cores do.
// conj(G) q is formed as conj(G conj(q)).
// SHARE: where the tiles would leave much of the card idle, `share` workgroups
// take the offsets of each half tile and store their sums in sorted order, and
// k_join_split adds them: a wavefront's offset takes 4 us, and one with four of
// them set the time of a 16^3 grid (product 22 us; with four workgroups 13 us
// and 4 us of join; the last workgroup adding the sums behind agent-scope fences
// instead took 21 us).
constexpr int kSplitWaves = 8;
constexpr int kSplitCols = kHelmSplitCols;

template <bool RED, bool CONJ, bool COMP, bool ONE, bool SHARE>
__global__ __launch_bounds__(64 * kSplitWaves) __attribute__((amdgpu_waves_per_eu(2))) void k_helm_split_cols(
    int key_bits, HelmTiles ht, HelmInline inl, int32_t nrhs, const int32_t *__restrict__ leaf_start,
    const uint64_t *__restrict__ leaf_key, const int32_t *__restrict__ perm,
    const int64_t *__restrict__ nbr_start, const int32_t *__restrict__ nbr_idx,
    const int64_t *__restrict__ red_start, const int64_t *__restrict__ red_row, const float2 *__restrict__ src,
    const u32x4 *__restrict__ blocks, int32_t copies, const float2 *__restrict__ zeros,
    const int32_t *__restrict__ inst_table, const float *__restrict__ inst_scale, const double *__restrict__ kh_dev,
    float2 *__restrict__ u, int32_t share, double2 *__restrict__ parts, int64_t entries) {
    using S = typename std::conditional<COMP, double, float>::type;
    __shared__ ColMap<kSplitCols> s_map;
    const ColMapView sm = s_map.view();
    // one right-hand side: until the sums, two tiles of Q rows in a wavefront's part
    __shared__ __attribute__((aligned(16))) S s_red[kSplitWaves][16][2][64];
    static_assert(sizeof(s_red[0]) >= 2 * 32 * 16 * sizeof(float2), "Q tiles do not fit");
    __shared__ float2 s_g[kDistances];
    const int tid = threadIdx.x, lane = tid & 63;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    int64_t item = p2pd::xcd_contiguous(blockIdx.x, gridDim.x);
    int part = 0;
    if constexpr (SHARE) {
        part = static_cast<int>(item % share);
        item /= share;
    }
    const int rt = static_cast<int>(item & 1);
    const ColTile ct = col_tile<kSplitCols>(inl, ht, nrhs, inst_table, inst_scale, nullptr,
                                            ht.tile0 + static_cast<int32_t>(item >> 1));
    const int col = lane & 31, half = lane >> 5;
    const ColLane cl = col_lane<ONE>(ct, nrhs, col);
    col_map<RED, 64 * kSplitWaves>(sm, key_bits, cl.A0, cl.boxes, leaf_start, leaf_key, nbr_start, nbr_idx, red_start,
                                   red_row);
    // the offsets that occur in this tile, as a bit mask
    const uint32_t present = static_cast<uint32_t>(__ballot(lane < 27 && sm.present[min(lane, 26)] != 0));
    const int n_off = __popc(present);
    // this wave's offsets: from the w0-th on every n_waves-th (n_off >= 1)
    const int n_waves = SHARE ? kSplitWaves * share : kSplitWaves, w0 = SHARE ? kSplitWaves * part + w : w;
    const int n_slots = n_off > w0 ? (n_off - w0 + n_waves - 1) / n_waves : 0;
    auto offset_of = [&](int slot) {   // the (w0 + n_waves slot)-th set bit, the last one past the end
        uint32_t m = present;
        const int k = min(w0 + n_waves * slot, n_off - 1);
        for (int i = 0; i < k; ++i) m &= m - 1;
        return __builtin_amdgcn_readfirstlane(__ffs(m) - 1);
    };
    const u32x4 *__restrict__ gtab =
        blocks + static_cast<int64_t>(ct.tab) * copies * kSplitTable + half * 6 * 64 + 32 * rt + col;
    // Sources at k-step ks: rows 16 ks + 8 half + 0..7 of this lane's column.  With
    // one right-hand side they are 64 bytes of a box's run, which lanes of
    // neighbouring columns would read at a stride of 512, a cache-line lookup
    // for every lane and 16 bytes; instead eight lanes read the 128 bytes of a
    // k-step of one column (lane / 8 of each of four groups of columns), and
    // the rows change lanes through LDS, 16-byte pieces of column c in the
    // order of the exclusive or with c / 2 (no bank conflicts).
    const float2 *qp[ONE ? 4 : 1];
    int64_t qs = 0;
    const u32x4 *gp = nullptr;
    float4 *const s_q = reinterpret_cast<float4 *>(&s_red[w][0][0][0]);   // [2][32 columns][8 pieces]
    const int piece = lane & 7;
    auto open = [&](int slot) {
        const int o = offset_of(slot);
        gp = gtab + o * 8 * 6 * 64;
        if constexpr (ONE) {
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int c = 8 * i + (lane >> 3);
                const int64_t row = sm.row[o * kSplitCols + c];
                qp[i] = (row >= 0 && c < ct.cnt ? src + row : zeros) + 2 * piece;
            }
        } else {
            const int64_t row = sm.row[o * kSplitCols + cl.box];
            qs = row >= 0 ? nrhs : 1;
            qp[0] = (row >= 0 ? src + row * nrhs : zeros) + 8 * half * qs + cl.rhs;
        }
    };
    auto load_q = [&](int ks, float (&v)[16]) {
        if constexpr (ONE) {
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const float4 x = *reinterpret_cast<const float4 *>(qp[i] + 16 * ks);
                v[4 * i] = x.x;
                v[4 * i + 1] = x.y;
                v[4 * i + 2] = x.z;
                v[4 * i + 3] = x.w;
            }
        } else {
            const float2 *q = qp[0] + 16 * ks * qs;
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                const float2 x = *q;
                v[2 * j] = x.x;
                v[2 * j + 1] = x.y;
                q += qs;
            }
        }
    };
    // one right-hand side: the loaded pieces to the lanes of their columns
    auto swap_q = [&](int buf, float (&v)[16]) {
        if constexpr (ONE) {
            float4 *d = s_q + buf * 256;
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int c = 8 * i + (lane >> 3);
                d[c * 8 + (piece ^ ((c >> 1) & 7))] = make_float4(v[4 * i], v[4 * i + 1], v[4 * i + 2], v[4 * i + 3]);
            }
            __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
            __builtin_amdgcn_wave_barrier();
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const float4 x = d[col * 8 + ((4 * half + j) ^ ((col >> 1) & 7))];
                v[4 * j] = x.x;
                v[4 * j + 1] = x.y;
                v[4 * j + 2] = x.z;
                v[4 * j + 3] = x.w;
            }
        }
    };
    auto load_g = [&](int ks, u32x4 (&g)[6]) {
#pragma unroll
        for (int p = 0; p < 6; ++p) g[p] = gp[(ks * 2 * 6 + p) * 64];
    };
    uint32_t nz[2] = {0, 0};   // the bits of every Re q and Im q
    // the h, m, l parts of Re q and Im q (negated with CONJ)
    auto split_q = [&](const float (&v)[16], u32x4 (&q)[6]) {
#pragma unroll
        for (int c = 0; c < 2; ++c)
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                float a = v[4 * j + c], b = v[4 * j + 2 + c];
                if (CONJ && c == 1) {
                    a = -a;
                    b = -b;
                }
                uint32_t h, m, l;
                split_pair(a, b, h, m, l, nz[c]);
                q[3 * c][j] = h;
                q[3 * c + 1][j] = m;
                q[3 * c + 2][j] = l;
            }
    };
    const floatx16 zero = floatx16{0};
    floatx16 pa = zero, pb = zero, pc = zero;   // sums of Re Re, Im Im, and Re Im + Im Re
    S cr[16], ci[16];
    if constexpr (COMP) {
#pragma unroll
        for (int r = 0; r < 16; ++r) cr[r] = ci[r] = 0.0;
    }
    auto mfma = [](const u32x4 &a, const u32x4 &b, const floatx16 &c) {
        return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c,
                                                       0, 0, 0);
    };
    auto mma = [&](const u32x4 (&g)[6], const u32x4 (&q)[6], bool fresh) {
#pragma unroll
        for (int p = 2; p >= 0; --p)
#pragma unroll
            for (int r = 2 - p; r >= 0; --r) {
                const bool f = fresh && p == 2;
                pa = mfma(g[p], q[r], f ? zero : pa);
                pc = mfma(g[p], q[3 + r], f ? zero : pc);
                pb = mfma(g[3 + p], q[3 + r], f ? zero : pb);
                pc = mfma(g[3 + p], q[r], pc);
            }
    };
    float raw[2][16];
    u32x4 g[2][6], q[6];
    if (n_slots > 0) {
        open(0);
        load_g(0, g[0]);
        load_q(0, raw[0]);
    }
    // the caller-order rows of the two targets this lane stores at the end
    int64_t dst[2] = {0, 0};
    if (col < ct.cnt) {
#pragma unroll
        for (int k = 0; k < 2; ++k) {
            const int r = 2 * w + k;
            const int32_t row = sm.tstart[cl.box] + 32 * rt + 8 * (r / 4) + 4 * half + r % 4;
            dst[k] = SHARE ? part * (entries / nrhs) + row : static_cast<int64_t>(perm[row]);
            if constexpr (!ONE) dst[k] = dst[k] * nrhs + cl.rhs;
        }
    }
    for (int slot = 0; slot < n_slots; ++slot) {
#pragma unroll
        for (int ks = 0; ks < 4; ++ks) {
            // the next k-step's operands (past the last offset the last one's again)
            if (ks == 3) open(slot + 1);
            load_q((ks + 1) & 3, raw[(ks + 1) & 1]);
            load_g((ks + 1) & 3, g[(ks + 1) & 1]);
            // without the barriers the scheduler sinks the loads to their uses
            __builtin_amdgcn_sched_barrier(0);
            swap_q(ks & 1, raw[ks & 1]);
            split_q(raw[ks & 1], q);
            mma(g[ks & 1], q, COMP && ks == 0);
            __builtin_amdgcn_sched_barrier(0);
        }
        if constexpr (COMP) {
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                cr[r] += static_cast<double>(pa[r] - pb[r]);
                ci[r] += static_cast<double>(pc[r]);
            }
        }
    }
    if constexpr (!COMP) {
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            cr[r] = pa[r] - pb[r];
            ci[r] = pc[r];
        }
    }
    const double kh = table_kh(inl, kh_dev, ct.tab);
    const bool again = sums_unheld<32>(kh, nz[0], nz[1], cr, ci);
#pragma unroll
    for (int r = 0; r < 16; ++r) {
        s_red[w][r][0][lane] = cr[r];
        s_red[w][r][1][lane] = ci[r];
    }
    if (again) {
        uint32_t offs = 0;
        for (int slot = 0; slot < n_slots; ++slot) offs |= 1u << offset_of(slot);
        const RedoSource f{sm.row + min(cl.box, cl.boxes - 1), kSplitCols, src, zeros, nrhs, cl.rhs, CONJ};
        redo_half_tile<S>(offs, kh, s_g, f, rt, &s_red[w][0][0][0]);
    }
    __syncthreads();
    if (col < ct.cnt) {
#pragma unroll
        for (int k = 0; k < 2; ++k) {
            const int r = 2 * w + k;
            S tr = s_red[0][r][0][lane], ti = s_red[0][r][1][lane];
#pragma unroll
            for (int v = 1; v < kSplitWaves; ++v) {
                tr += s_red[v][r][0][lane];
                ti += s_red[v][r][1][lane];
            }
            if (CONJ) ti = -ti;
            if constexpr (SHARE)
                parts[dst[k]] = make_double2(static_cast<double>(tr * ct.sc), static_cast<double>(ti * ct.sc));
            else
                u[dst[k]] = make_float2(static_cast<float>(tr * ct.sc), static_cast<float>(ti * ct.sc));
        }
    }
}

// The sums of the workgroups that share a half tile, in order, to caller order.
__global__ __launch_bounds__(256) void k_join_split(const double2 *__restrict__ parts, int32_t share,
                                                    const int32_t *__restrict__ perm, int64_t entries, int32_t nrhs,
                                                    float2 *__restrict__ u) {
    const int64_t e = static_cast<int64_t>(blockIdx.x) * 256 + threadIdx.x;
    if (e >= entries) return;
    const int64_t row = e / nrhs;
    const int64_t d = static_cast<int64_t>(perm[row]) * nrhs + (e - row * nrhs);
    double2 s = parts[e];
    for (int p = 1; p < share; ++p) {
        const double2 v = parts[p * entries + e];
        s.x += v.x;
        s.y += v.y;
    }
    u[d] = make_float2(static_cast<float>(s.x), static_cast<float>(s.y));
}

// ------------------------------------------------------------ many columns --
// The same product when there are columns enough to fill the card: a workgroup
// of 2 W wavefronts takes W tiles of 32 columns through the offsets together,
// so that a G block is read from L2 once for 32 W columns and its operands come
// from LDS.  A wavefront holds all 64 targets of 16 columns
// (v_mfma_f32_16x16x32_bf16): each Q value is then split once per target box,
// and 32 accumulator and 64 FP64-sum registers leave room for two wavefronts
// per SIMD, one of which splits, adds and waits while the other multiplies.
// On the 128-grid, 64-RHS batch the product takes 22.0 ms, 1.20 PFLOP/s of BF16
// products (FP32 matrix instructions: 26.4 ms); under the profiler the matrix cores
// are busy 0.60 of the cycles at 1.71 GHz.  Compared at 20.8 ms, before the checks
// of the sums: a wavefront per SIMD with 64 x 32 results and three real products
// per complex one issues a quarter fewer matrix instructions, but its vector work,
// eight instructions per matrix instruction, hides behind nothing: 22.3 ms.  Row
// tiles of 32 over twice the wavefronts split every Q value twice: 24.1 ms.
// G is staged 32 sources at a time through three LDS buffers: the stage after
// next is written behind a stage's one barrier and its loads are issued a stage
// earlier, so a barrier waits for the slowest wavefront only.  The barrier
// stands at the middle of the stage for the first W wavefronts and at its start
// for the others, so that the two of a SIMD do not split at the same time
// (21.6 ms with all at the middle, 20.8 so).  G parts are read from LDS two plane pairs
// ahead of their products.
// Items (one tile, or two with 64 right-hand sides per wave) are taken in tree
// order from eight queues, one per XCD over a contiguous eighth of them
// (neighbouring boxes meet in one XCD's L2), a workgroup whose own queue is
// empty taking from the others in turn; counters only grow, so every workgroup
// ends after at most eight misses.
constexpr int kWideStage = 4 * 6 * 64;    // 16-byte operands of a stage: [run of eight sources][plane][target]

typedef __amdgpu_buffer_rsrc_t Rsrc;
template <int W, bool RED, bool CONJ, bool COMP, bool UNI>
__global__ __launch_bounds__(128 * W) __attribute__((amdgpu_waves_per_eu(2))) void k_helm_split(
    int key_bits, HelmTiles ht, HelmInline inl, int32_t nrhs, int32_t n_tiles, int32_t per_item, int32_t cap,
    const int32_t *__restrict__ leaf_start, const uint64_t *__restrict__ leaf_key, const int32_t *__restrict__ perm,
    const int64_t *__restrict__ nbr_start, const int32_t *__restrict__ nbr_idx,
    const int64_t *__restrict__ red_start, const int64_t *__restrict__ red_row, const float2 *__restrict__ src,
    const u32x4 *__restrict__ blocks, int32_t copies, const float2 *__restrict__ zeros,
    const int32_t *__restrict__ inst_table, const float *__restrict__ inst_scale, const double *__restrict__ kh_dev,
    int32_t *__restrict__ counter, float2 *__restrict__ u) {
    using S = typename std::conditional<COMP, double, float>::type;
    constexpr int NT = 128 * W, NL = kWideStage / NT;
    extern __shared__ __attribute__((aligned(16))) char smem[];
    __shared__ int32_t s_item;
    __shared__ float2 s_g[kDistances];
    u32x4 *const sg = reinterpret_cast<u32x4 *>(smem);
    const ColMapView sm = col_map_view(smem + 3 * kWideStage * sizeof(u32x4), cap);
    const int tid = threadIdx.x, lane = tid & 63, col = lane & 15, kq = lane >> 4;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int xcd = static_cast<int>(blockIdx.x & 7);
    const int64_t items = (n_tiles + per_item - 1) / per_item;
    auto slice = [&](int x) { return items * x / 8; };
    // thread 0: the next ticket is drawn at the start of an item and looked at after
    // it while its queue holds more items than there are workgroups to an XCD;
    // towards the end it would keep an item from a workgroup that is free sooner (a
    // launch of 203 items by 203 workgroups took two rounds, 260 us instead of 150)
    int sl = 0;
    bool drawn = true;
    int32_t ticket = tid == 0 ? atomicAdd(&counter[xcd], 1) : 0;
    for (;;) {
        if (tid == 0) {
            int32_t it = -1;
            if (!drawn) ticket = atomicAdd(&counter[(xcd + sl) & 7], 1);
            for (;;) {
                const int x = (xcd + sl) & 7;
                if (slice(x) + ticket < slice(x + 1)) {
                    it = static_cast<int32_t>(slice(x) + ticket);
                    break;
                }
                if (++sl == 8) break;
                ticket = atomicAdd(&counter[(xcd + sl) & 7], 1);
            }
            s_item = it;
        }
        __syncthreads();
        const int32_t item = __builtin_amdgcn_readfirstlane(s_item);
        if (item < 0) break;
        if (tid == 0) {
            drawn = slice(((xcd + sl) & 7) + 1) - item > gridDim.x / 8 + 1;
            if (drawn) ticket = atomicAdd(&counter[(xcd + sl) & 7], 1);
        }
        const int32_t tile_end = static_cast<int32_t>(min<int64_t>((item + int64_t(1)) * per_item, n_tiles));
        for (int32_t tile = item * per_item; tile < tile_end; ++tile) {
            const ColTile ct = col_tile<32 * W>(inl, ht, nrhs, inst_table, inst_scale, nullptr, ht.tile0 + tile);
            const ColLane cl = col_lane<false>(ct, nrhs, 16 * w + col);
            __syncthreads();   // the map and the stages of the tile before are no longer read
            col_map<RED, NT>(sm, key_bits, cl.A0, cl.boxes, leaf_start, leaf_key, nbr_start, nbr_idx, red_start,
                             red_row);
            uint32_t present = static_cast<uint32_t>(__ballot(lane < 27 && sm.present[min(lane, 26)] != 0));
            if (present == 0) present = 1;   // empty lists: one offset, every source row absent
            const int n_off = __popc(present);
            const int64_t copy = (blockIdx.x >> 3) % copies;   // the workgroups of one XCD spread over the copies
            const u32x4 *__restrict__ gtab =
                blocks + (static_cast<int64_t>(ct.tab) * copies + copy) * kSplitTable + tid;

            // stages: two per offset that occurs, in order; past the end the last offset's again
            u32x4 st[NL];
            uint32_t lm = present;
            int lh = 0;
            auto load_stage = [&]() {
                const u32x4 *p = gtab + ((__ffs(lm) - 1) * 2 + lh) * kWideStage;
#pragma unroll
                for (int i = 0; i < NL; ++i) st[i] = p[i * NT];
                lh ^= 1;
                if (lh == 0 && (lm & (lm - 1))) lm &= lm - 1;
            };
            auto write_stage = [&](int buf) {
#pragma unroll
                for (int i = 0; i < NL; ++i) sg[buf * kWideStage + i * NT + tid] = st[i];
            };
            // this lane's source rows at an offset.  UNI: the wavefront's columns are
            // 16 right-hand sides of one box, so the rows are reached through a
            // buffer descriptor (scalar registers; of length zero where the box has
            // no such neighbour: such loads return zeros), a fixed lane offset and a
            // scalar offset per row, without vector instructions on addresses.
            // Otherwise a pointer and row stride per lane.
            const float2 *qp = nullptr;
            int64_t qs = 0;
            Rsrc qr_;
            const int rhs0 = __builtin_amdgcn_readfirstlane(uni_first_rhs(cl.rhs));
            const int voff = (8 * kq * nrhs + col) * static_cast<int>(sizeof(float2));
            auto rows_of = [&](int o) {
                const int64_t row = sm.row[o * cap + cl.box];
                if constexpr (UNI) {
                    const int64_t r = (static_cast<int64_t>(__builtin_amdgcn_readfirstlane(static_cast<int>(row >> 32))) << 32) |
                                      static_cast<uint32_t>(__builtin_amdgcn_readfirstlane(static_cast<int>(row)));
                    qr_ = __builtin_amdgcn_make_buffer_rsrc(
                        const_cast<float2 *>(src + (r >= 0 ? r * nrhs : 0) + rhs0), 0,
                        r >= 0 ? (64 * nrhs - rhs0) * static_cast<int>(sizeof(float2)) : 0, 0x00020000);
                } else {
                    qs = row >= 0 ? nrhs : 1;
                    qp = (row >= 0 ? src + row * nrhs : zeros) + 8 * kq * qs + cl.rhs;
                }
            };
            auto load_q = [&](int ks, float (&v)[16]) {
                const float2 *p = qp + 32 * ks * qs;
#pragma unroll
                for (int j = 0; j < 8; ++j) {
                    float2 x;
                    if constexpr (UNI) {
                        x = __builtin_bit_cast(float2, __builtin_amdgcn_raw_buffer_load_b64(
                                                           qr_, voff, (32 * ks + j) * nrhs * static_cast<int>(sizeof(float2)), 0));
                    } else {
                        x = *p;
                        p += qs;
                    }
                    v[2 * j] = x.x;
                    v[2 * j + 1] = x.y;
                }
            };
            uint32_t nz_r = 0, nz_i = 0;   // the bits of every Re q and Im q
            // parts of Re q, Im q and -Im q
            auto split_q = [&](const float (&v)[16], u32x4 (&qr)[3], u32x4 (&qi)[3], u32x4 (&qn)[3]) {
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    uint32_t h, m, l;
                    split_pair(v[4 * j], v[4 * j + 2], h, m, l, nz_r);
                    qr[0][j] = h;
                    qr[1][j] = m;
                    qr[2][j] = l;
                    split_pair(v[4 * j + 1], v[4 * j + 3], h, m, l, nz_i);
                    qi[0][j] = h;
                    qi[1][j] = m;
                    qi[2][j] = l;
                }
#pragma unroll
                for (int p = 0; p < 3; ++p) qn[p] = qi[p] ^ 0x80008000u;
            };
            // the pairs of planes (part of Re G, the same part of Im G) of a stage
            // in the order of their use, l, m, h of row tile 0, then of 1, ...
            auto read_g = [&](int buf, int pair, u32x4 (&g)[2]) {
                const int rt = pair / 3, p = 2 - pair % 3;
#pragma unroll
                for (int c = 0; c < 2; ++c) g[c] = sg[buf * kWideStage + (kq * 6 + 3 * c + p) * 64 + 16 * rt + col];
            };
            floatx4 re[4], im[4];
            const floatx4 zero = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int rt = 0; rt < 4; ++rt) re[rt] = im[rt] = zero;
            // the sums over the offsets, each offset's products starting anew
            S cr[16], ci[16];
#pragma unroll
            for (int r = 0; r < 16; ++r) cr[r] = ci[r] = 0;
            auto mfma = [](const u32x4 &x, const u32x4 &y, const floatx4 &c) {
                return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, x),
                                                               __builtin_bit_cast(bf16x8, y), c, 0, 0, 0);
            };

            float raw[16];
            u32x4 g[3][2];
            load_stage();
            write_stage(0);
            load_stage();
            write_stage(1);
            load_stage();
            const bool late = w >= W;   // the second wavefront of a SIMD
            uint32_t cm = present;
            rows_of(__ffs(cm) - 1);
            load_q(0, raw);
            __syncthreads();
            read_g(0, 0, g[0]);
            read_g(0, 1, g[1]);
            int b0 = 0, b1 = 1, b2 = 2;   // buffers of this stage, the next and the one after
            auto next_stage = [&]() {
                __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
                __builtin_amdgcn_s_barrier();
                __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
                write_stage(b2);
                load_stage();
            };
            for (int k = 0; k < n_off; ++k) {
#pragma unroll
                for (int ks = 0; ks < 2; ++ks) {
                    if (late) next_stage();
                    u32x4 qr[3], qi[3], qn[3];
                    split_q(raw, qr, qi, qn);
                    __builtin_amdgcn_sched_barrier(0);
                    if (ks == 1) {
                        if (cm & (cm - 1)) cm &= cm - 1;
                        rows_of(__ffs(cm) - 1);
                    }
                    load_q(1 - ks, raw);   // the next stage's
#pragma unroll
                    for (int rt = 0; rt < 4; ++rt) {
                        if (rt == 2 && !late) next_stage();
                        // conj(G) q = conj(G conj(q))
                        const u32x4(&qa)[3] = CONJ ? qn : qi, (&qb)[3] = CONJ ? qi : qn;
#pragma unroll
                        for (int p = 2; p >= 0; --p) {
                            const int pair = 3 * rt + 2 - p, ahead = pair + 2;
                            read_g(ahead < 12 ? b0 : b1, ahead % 12, g[ahead % 3]);
                            __builtin_amdgcn_sched_barrier(0);
                            const u32x4(&gc)[2] = g[pair % 3];
#pragma unroll
                            for (int r = 2 - p; r >= 0; --r) {
                                const bool fresh = ks == 0 && p == 2;
                                re[rt] = mfma(gc[0], qr[r], fresh ? zero : re[rt]);
                                im[rt] = mfma(gc[0], qa[r], fresh ? zero : im[rt]);
                                re[rt] = mfma(gc[1], qb[r], re[rt]);
                                im[rt] = mfma(gc[1], qr[r], im[rt]);
                            }
                            __builtin_amdgcn_sched_barrier(0);
                        }
                    }
                    const int t = b0;
                    b0 = b1;
                    b1 = b2;
                    b2 = t;
                }
#pragma unroll
                for (int rt = 0; rt < 4; ++rt)
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        cr[4 * rt + r] += static_cast<S>(re[rt][r]);
                        ci[4 * rt + r] += static_cast<S>(im[rt][r]);
                    }
            }
            const double kh = table_kh(inl, kh_dev, ct.tab);
            const bool again = sums_unheld<16>(kh, nz_r, nz_i, cr, ci);
            const bool mine = 16 * w + col < ct.cnt;
            const int32_t *const row_of = perm + sm.tstart[cl.box];
            if (again) {
                const RedoSource f{sm.row + cl.box, cap, src, zeros, nrhs, cl.rhs, CONJ};
                redo_columns(present, kh, s_g, f, mine, row_of, ct.sc, u);
            } else if (mine) {
#pragma unroll
                for (int rt = 0; rt < 4; ++rt)
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        const int64_t at = static_cast<int64_t>(row_of[16 * rt + 4 * kq + r]) * nrhs + cl.rhs;
                        const float x = static_cast<float>(cr[4 * rt + r] * ct.sc),
                                    y = static_cast<float>(ci[4 * rt + r] * ct.sc);
                        u[at] = make_float2(x, CONJ ? -y : y);
                    }
            }
        }
        __syncthreads();   // s_item has been read by all
    }
}

__global__ void k_zero_counter(int32_t *c, int n) {
    if (static_cast<int>(threadIdx.x) < n) c[threadIdx.x] = 0;
}

}  // namespace

p2p_status launch_split_prep(const double *d_kh, const HelmInline &inl, int32_t n_tables, int32_t copies,
                             int32_t nrhs, void *blocks, const void *q, const int32_t *perm, int64_t n, void *sorted,
                             hipStream_t s) {
    const int64_t g_wgs = static_cast<int64_t>(n_tables) * kSplitTableWgs;
    const uint64_t units = sorted ? static_cast<uint64_t>(n) * static_cast<uint64_t>(nrhs) : 0;
    if (units > INT32_MAX) return fail(P2P_EINVAL, "too many entries for the product of few columns");
    const int64_t wgs = g_wgs + static_cast<int64_t>((units + kPermuteEntries - 1) / kPermuteEntries);
    if (wgs == 0) return P2P_OK;
    k_split_prep<<<static_cast<unsigned>(wgs), 256, 0, s>>>(
        d_kh, inl, n_tables, copies, nrhs, static_cast<u32x4 *>(blocks), static_cast<int32_t>(g_wgs),
        static_cast<const float2 *>(q), perm, static_cast<uint32_t>(units), static_cast<float2 *>(sorted));
    P2P_LAUNCH_CHECK();
    return P2P_OK;
}

template <bool R, bool C, bool M, bool O>
static void launch_split(const HelmholtzMfmaArgs &a, const HelmTiles &ht, const HelmInline &inl, int32_t n_tiles,
                         hipStream_t s) {
    const int32_t share = a.parts ? helm_split_share(n_tiles) : 1;
    const int64_t entries = a.n * a.nrhs;
    const unsigned grid = 2u * static_cast<unsigned>(n_tiles) * static_cast<unsigned>(share);
#define P2P_SPLIT(SH)                                                                                           \
    k_helm_split_cols<R, C, M, O, SH><<<grid, 64 * kSplitWaves, 0, s>>>(                                        \
        a.key_bits, ht, inl, a.nrhs, a.leaf_start, a.leaf_key, a.perm, a.nbr_start, a.nbr_idx, a.red_start,     \
        a.red_row, a.src, reinterpret_cast<const u32x4 *>(a.blocks), a.copies, a.zeros, a.inst_table,           \
        a.inst_scale, a.kh, a.u, share, a.parts, entries)
    if (share > 1) {
        P2P_SPLIT(true);
        k_join_split<<<grid_for(entries, 256), 256, 0, s>>>(a.parts, share, a.perm, entries, a.nrhs, a.u);
    } else {
        P2P_SPLIT(false);
    }
#undef P2P_SPLIT
}

template <bool R, bool C, bool M>
static void launch_split(const HelmholtzMfmaArgs &a, const HelmTiles &ht, const HelmInline &inl, int32_t n_tiles,
                         hipStream_t s) {
    // one right-hand side: a box's rows are read 16 bytes at a time where they are aligned to that
    if (a.nrhs == 1 && (reinterpret_cast<uintptr_t>(a.src) & 15) == 0)
        launch_split<R, C, M, true>(a, ht, inl, n_tiles, s);
    else
        launch_split<R, C, M, false>(a, ht, inl, n_tiles, s);
}

p2p_status launch_helmholtz_split_cols(const HelmholtzMfmaArgs &a, const HelmTiles &ht, const HelmInline &inl,
                                       int32_t n_tiles, bool redundant, hipStream_t s) {
    if (n_tiles <= 0) return P2P_OK;
    const bool cj = a.conj != 0;
#define P2P_SPLIT_M(R, C) \
    if (a.comp) launch_split<R, C, true>(a, ht, inl, n_tiles, s); else launch_split<R, C, false>(a, ht, inl, n_tiles, s)
    if (redundant) { if (cj) { P2P_SPLIT_M(true, true); } else { P2P_SPLIT_M(true, false); } }
    else { if (cj) { P2P_SPLIT_M(false, true); } else { P2P_SPLIT_M(false, false); } }
#undef P2P_SPLIT_M
    P2P_LAUNCH_CHECK();
    return P2P_OK;
}

template <int W, bool R, bool C, bool M, bool U>
static p2p_status launch_wide(const HelmholtzMfmaArgs &a, const HelmTiles &ht, const HelmInline &inl,
                              int32_t n_tiles, int32_t per_item, unsigned grid, hipStream_t s) {
    // boxes a tile of 32 W columns can touch
    const int32_t cap = static_cast<int32_t>(std::min<int64_t>(32 * W, (32 * W + static_cast<int64_t>(a.nrhs) - 2) / a.nrhs + 1));
    constexpr size_t ring = 3 * kWideStage * sizeof(u32x4);
    const size_t lds = ring + col_map_bytes(cap);
    auto *k = k_helm_split<W, R, C, M, U>;
    // the largest a launch can need: the attribute belongs to the kernel, and threads
    // with other right-hand sides set it between each other's set and launch
    P2P_HIP(hipFuncSetAttribute(reinterpret_cast<const void *>(k), hipFuncAttributeMaxDynamicSharedMemorySize,
                                static_cast<int>(ring + col_map_bytes(32 * W))));
    k<<<grid, 128 * W, lds, s>>>(a.key_bits, ht, inl, a.nrhs, n_tiles, per_item, cap, a.leaf_start, a.leaf_key, a.perm,
                                a.nbr_start, a.nbr_idx, a.red_start, a.red_row, a.src,
                                reinterpret_cast<const u32x4 *>(a.blocks), a.copies, a.zeros, a.inst_table,
                                a.inst_scale, a.kh, a.counter, a.u);
    P2P_LAUNCH_CHECK();
    return P2P_OK;
}

template <int W, bool R, bool C>
static p2p_status launch_wide_m(const HelmholtzMfmaArgs &a, const HelmTiles &ht, const HelmInline &inl,
                                int32_t n_tiles, int32_t per_item, unsigned grid, hipStream_t s) {
    // 16 right-hand sides of one box per wavefront, a box's rows within 32-bit byte offsets
    const bool uni = a.nrhs % 16 == 0 && a.nrhs <= (1 << 20);
    if (a.comp)
        return uni ? launch_wide<W, R, C, true, true>(a, ht, inl, n_tiles, per_item, grid, s)
                   : launch_wide<W, R, C, true, false>(a, ht, inl, n_tiles, per_item, grid, s);
    return uni ? launch_wide<W, R, C, false, true>(a, ht, inl, n_tiles, per_item, grid, s)
               : launch_wide<W, R, C, false, false>(a, ht, inl, n_tiles, per_item, grid, s);
}

template <int W>
static p2p_status launch_wide_w(const HelmholtzMfmaArgs &a, const HelmTiles &ht, const HelmInline &inl,
                                int32_t n_tiles, int32_t per_item, unsigned grid, bool redundant, hipStream_t s) {
    const bool cj = a.conj != 0;
    if (redundant)
        return cj ? launch_wide_m<W, true, true>(a, ht, inl, n_tiles, per_item, grid, s)
                  : launch_wide_m<W, true, false>(a, ht, inl, n_tiles, per_item, grid, s);
    return cj ? launch_wide_m<W, false, true>(a, ht, inl, n_tiles, per_item, grid, s)
              : launch_wide_m<W, false, false>(a, ht, inl, n_tiles, per_item, grid, s);
}

p2p_status launch_helmholtz_split(const HelmholtzMfmaArgs &a, const HelmTiles &ht, const HelmInline &inl,
                                  int32_t n_tiles, bool redundant, int tiles_per_wg, int wg_per_cu, int rhs_tile,
                                  hipStream_t s) {
    if (n_tiles <= 0) return P2P_OK;
    int dev = 0, cus = 0;
    P2P_HIP(hipGetDevice(&dev));
    P2P_HIP(hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev));
    k_zero_counter<<<1, 64, 0, s>>>(a.counter, 8);
    P2P_LAUNCH_CHECK();
    const int32_t per_item = rhs_tile / 32;
    const int64_t items = (static_cast<int64_t>(n_tiles) + per_item - 1) / per_item;
    const unsigned grid = static_cast<unsigned>(std::min<int64_t>(items, static_cast<int64_t>(cus) * wg_per_cu));
    return tiles_per_wg == 2 ? launch_wide_w<2>(a, ht, inl, n_tiles, per_item, grid, redundant, s)
                             : launch_wide_w<4>(a, ht, inl, n_tiles, per_item, grid, redundant, s);
}

}  // namespace p2p
