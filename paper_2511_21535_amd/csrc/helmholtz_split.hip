// Near-field Helmholtz in single precision on the BF16 matrix cores, without
// giving up single precision: every FP32 operand is the exact sum of three
// BF16 values, x = h + m + l (8 significand bits each, the exponent range of
// FP32), and a real product takes the six partial products of order up to two,
// h h, h m, m h, m m, h l, l h, accumulated in FP32 by
// v_mfma_f32_32x32x16_bf16.  What is left out (m l, l m, l l) lies below
// 2^-23 of the product, as one FP32 rounding does, while the sixteen terms an
// instruction adds are rounded once instead of eight times: the error against
// 64 bits of a 64^3 grid is 1.8e-7 where FP32 matrix instructions (three real
// products per complex one) leave 2.2e-7.  A BF16 product takes a sixteenth of
// the FP32 one's time, so six cost 0.38 of it.  Magnitudes below about 1e-33
// lose their low parts to the subnormal range; infinities and NaN give NaN.
#include <type_traits>

#include "helm_columns.h"

namespace p2p {
namespace {

typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float floatx16 __attribute__((ext_vector_type(16)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

__device__ inline uint32_t bf16_pair(float a, float b) {
    const bf16x2 v = {static_cast<__bf16>(a), static_cast<__bf16>(b)};
    return __builtin_bit_cast(uint32_t, v);
}
__device__ inline float bf16_lo(uint32_t v) { return __uint_as_float(v << 16); }
__device__ inline float bf16_hi(uint32_t v) { return __uint_as_float(v & 0xffff0000u); }

// Two values into their three BF16 parts, packed in pairs.  Each difference is
// exact: what is left after rounding to 8 bits fits in the remaining 16.
__device__ inline void split_pair(float a, float b, uint32_t &h, uint32_t &m, uint32_t &l) {
    h = bf16_pair(a, b);
    const float a1 = a - bf16_lo(h), b1 = b - bf16_hi(h);
    m = bf16_pair(a1, b1);
    l = bf16_pair(a1 - bf16_lo(m), b1 - bf16_hi(m));
}

// G blocks of the split product.  For table t, copy c, box offset o, k-step ks
// (16 sources) and row tile rt (32 targets), np planes of 64 lanes x 16 bytes:
// lane l holds the eight sources 16 ks + 8 (l / 32) + 0..7 of target
// 32 rt + l % 32, the operand order of the instruction.  Planes: the h, m and l
// parts of Re G, of Im G and, with np = 9, of Re G + Im G (formed in double and
// rounded to single once, as Re and Im are).  64 zero float2 entries follow
// (the sources of an absent neighbour).  G depends on the squared distance
// alone, so a workgroup forms the 148 values it can take once, in double.
__global__ __launch_bounds__(256) void k_split_blocks(const double *__restrict__ kh_dev, HelmInline inl,
                                                      int32_t n_tables, int32_t copies, int32_t np,
                                                      u32x4 *__restrict__ out) {
    __shared__ float2 s_g[kDistances];
    __shared__ float s_sum[kDistances];
    constexpr int per = 27 * 4 * 2 * 64;            // lanes per table
    constexpr int wgs = per / 256;
    const int tab = static_cast<int>(blockIdx.x) / wgs;
    const int tid = threadIdx.x;
    if (tid < kDistances) {
        const double2 v = green(table_kh(inl, kh_dev, tab), tid);
        s_g[tid] = make_float2(static_cast<float>(v.x), static_cast<float>(v.y));
        s_sum[tid] = static_cast<float>(v.x + v.y);
    }
    __syncthreads();
    const int t = (static_cast<int>(blockIdx.x) % wgs) * 256 + tid;
    const int lane = t & 63, rt = (t >> 6) & 1, ks = (t >> 7) & 3, o = t >> 9;
    const int i = 32 * rt + (lane & 31), s0 = 16 * ks + 8 * (lane >> 5);
    float v[3][8];
#pragma unroll
    for (int j = 0; j < 8; ++j) {
        const int dd = near_distance(o, s0 + j, i);
        v[0][j] = s_g[dd].x;
        v[1][j] = s_g[dd].y;
        v[2][j] = s_sum[dd];
    }
    for (int c = 0; c < copies; ++c) {
        u32x4 *w = out + (static_cast<int64_t>(tab) * copies + c) * (27 * 8) * np * 64 +
                   static_cast<int64_t>((o * 4 + ks) * 2 + rt) * np * 64 + lane;
#pragma unroll
        for (int q = 0; q < 3; ++q) {
            if (3 * q >= np) break;
            u32x4 h, m, l;
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                uint32_t hh, mm, ll;
                split_pair(v[q][2 * j], v[q][2 * j + 1], hh, mm, ll);
                h[j] = hh;
                m[j] = mm;
                l[j] = ll;
            }
            w[(3 * q) * 64] = h;
            w[(3 * q + 1) * 64] = m;
            w[(3 * q + 2) * 64] = l;
        }
    }
    if (blockIdx.x == 0 && tid < 32)
        out[static_cast<int64_t>(n_tables) * copies * (27 * 8) * np * 64 + tid] = u32x4{0, 0, 0, 0};
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
constexpr int kSplitWaves = 8;
constexpr int kSplitCols = kHelmSplitCols;

template <bool RED, bool CONJ, bool COMP, bool ONE>
__global__ __launch_bounds__(64 * kSplitWaves) __attribute__((amdgpu_waves_per_eu(2))) void k_helm_split_cols(
    int key_bits, HelmTiles ht, HelmInline inl, int32_t nrhs, const int32_t *__restrict__ leaf_start,
    const uint64_t *__restrict__ leaf_key, const int32_t *__restrict__ perm,
    const int64_t *__restrict__ nbr_start, const int32_t *__restrict__ nbr_idx,
    const int64_t *__restrict__ red_start, const int64_t *__restrict__ red_row, const float2 *__restrict__ src,
    const u32x4 *__restrict__ blocks, int32_t np, int32_t copies, const float2 *__restrict__ zeros,
    const int32_t *__restrict__ inst_table, const float *__restrict__ inst_scale, float2 *__restrict__ u) {
    using S = typename std::conditional<COMP, double, float>::type;
    __shared__ ColMap<kSplitCols> sm;
    __shared__ S s_red[kSplitWaves][16][2][64];
    const int tid = threadIdx.x, lane = tid & 63;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int64_t item = p2pd::xcd_contiguous(blockIdx.x, gridDim.x);
    const int rt = static_cast<int>(item & 1);
    const ColTile ct = col_tile<kSplitCols>(inl, ht, nrhs, inst_table, inst_scale, nullptr,
                                            static_cast<int32_t>(item >> 1));
    const int col = lane & 31, half = lane >> 5;
    const ColLane cl = col_lane<ONE>(ct, nrhs, col);
    col_map<RED, kSplitCols, 64 * kSplitWaves>(sm, key_bits, cl.A0, cl.boxes, leaf_start, leaf_key, nbr_start,
                                               nbr_idx, red_start, red_row);
    // the offsets that occur in this tile, as a bit mask
    const uint32_t present = static_cast<uint32_t>(__ballot(lane < 27 && sm.present[min(lane, 26)] != 0));
    const int n_off = __popc(present);
    const int n_slots = (n_off - w + kSplitWaves - 1) / kSplitWaves;   // this wave's offsets (n_off >= 1)
    auto offset_of = [&](int slot) {   // the (w + 8 slot)-th set bit, the last one past the end
        uint32_t m = present;
        const int k = min(w + kSplitWaves * slot, n_off - 1);
        for (int i = 0; i < k; ++i) m &= m - 1;
        return __builtin_amdgcn_readfirstlane(__ffs(m) - 1);
    };
    const u32x4 *__restrict__ gtab =
        blocks + static_cast<int64_t>(ct.tab) * copies * (27 * 8) * np * 64 + static_cast<int64_t>(rt) * np * 64 + lane;
    // this lane's sources at k-step ks: rows 16 ks + 8 half + 0..7 of its column
    const float2 *qp = nullptr;
    int64_t qs = 0;
    const u32x4 *gp = nullptr;
    auto open = [&](int slot) {
        const int o = offset_of(slot);
        const int64_t row = sm.row[o][cl.box];
        gp = gtab + static_cast<int64_t>(o) * 8 * np * 64;
        if constexpr (ONE) {
            qp = (row >= 0 && col < ct.cnt ? src + row : zeros) + 8 * half;
        } else {
            qp = row >= 0 ? src + (row + 8 * half) * nrhs + cl.rhs : zeros;
            qs = row >= 0 ? nrhs : 0;
        }
    };
    auto load_q = [&](int ks, float (&v)[16]) {
        if constexpr (ONE) {
            const float4 *q4 = reinterpret_cast<const float4 *>(qp + 16 * ks);
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const float4 x = q4[j];
                v[4 * j] = x.x;
                v[4 * j + 1] = x.y;
                v[4 * j + 2] = x.z;
                v[4 * j + 3] = x.w;
            }
        } else {
            const float2 *q = qp + 16 * ks * qs;
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                const float2 x = *q;
                v[2 * j] = x.x;
                v[2 * j + 1] = x.y;
                q += qs;
            }
        }
    };
    auto load_g = [&](int ks, u32x4 (&g)[6]) {
#pragma unroll
        for (int p = 0; p < 6; ++p) g[p] = gp[(ks * 2 * np + p) * 64];
    };
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
                split_pair(a, b, h, m, l);
                q[3 * c][j] = h;
                q[3 * c + 1][j] = m;
                q[3 * c + 2][j] = l;
            }
    };
    const floatx16 zero = floatx16{0};
    floatx16 pa = zero, pb = zero, pc = zero;   // sums of Re Re, Im Im, and Re Im + Im Re
    constexpr int CN = COMP ? 16 : 1;
    double cr[CN], ci[CN];
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
            dst[k] = perm[sm.tstart[cl.box] + 32 * rt + 8 * (r / 4) + 4 * half + r % 4];
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
#pragma unroll
    for (int r = 0; r < 16; ++r) {
        if constexpr (COMP) {
            s_red[w][r][0][lane] = cr[r];
            s_red[w][r][1][lane] = ci[r];
        } else {
            s_red[w][r][0][lane] = pa[r] - pb[r];
            s_red[w][r][1][lane] = pc[r];
        }
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
            u[dst[k]] = make_float2(static_cast<float>(tr * ct.sc), static_cast<float>(ti * ct.sc));
        }
    }
}

}  // namespace

p2p_status launch_split_blocks(const double *d_kh, const HelmInline &inl, int32_t n_tables, int32_t copies,
                               int32_t planes, void *blocks, hipStream_t s) {
    const int64_t wgs = static_cast<int64_t>(n_tables) * (27 * 4 * 2 * 64 / 256);
    k_split_blocks<<<static_cast<unsigned>(wgs), 256, 0, s>>>(d_kh, inl, n_tables, copies, planes,
                                                             static_cast<u32x4 *>(blocks));
    P2P_LAUNCH_CHECK();
    return P2P_OK;
}

template <bool R, bool C, bool M>
static void launch_split(const HelmholtzMfmaArgs &a, const HelmTiles &ht, const HelmInline &inl, int32_t n_tiles,
                         hipStream_t s) {
    const unsigned grid = 2u * static_cast<unsigned>(n_tiles);
#define P2P_SPLIT(O)                                                                                            \
    k_helm_split_cols<R, C, M, O><<<grid, 64 * kSplitWaves, 0, s>>>(                                            \
        a.key_bits, ht, inl, a.nrhs, a.leaf_start, a.leaf_key, a.perm, a.nbr_start, a.nbr_idx, a.red_start,      \
        a.red_row, a.src, reinterpret_cast<const u32x4 *>(a.blocks), a.planes, a.copies, a.zeros, a.inst_table,  \
        a.inst_scale, a.u)
    // one right-hand side: a lane's eight sources are one 64-byte run, read 16
    // bytes at a time where the rows are aligned to that
    if (a.nrhs == 1 && (reinterpret_cast<uintptr_t>(a.src) & 15) == 0) P2P_SPLIT(true); else P2P_SPLIT(false);
#undef P2P_SPLIT
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

}  // namespace p2p
