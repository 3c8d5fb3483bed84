// Near-field Helmholtz sum in double on the FP64 matrix cores, the (target box,
// right-hand side) pairs as the columns of the product (the dense regular case
// of Sec. 5.1).  Kept in a file of its own: it is compiled with the matrix
// accumulators in ordinary vector registers (-amdgpu-mfma-vgpr-form).
#include "helm_columns.h"

namespace p2p {
namespace {

// A column is a (target box, right-hand side) pair: on a regular grid G_o
// depends only on the box offset o, so boxes and right-hand sides are alike to
// the product.  For a tile of up to 16 consecutive columns (b_j, r_j) of one
// instance, numbered box * nrhs + rhs,
//     U (64 x 16) = sum_o G_o (64 x 64) Q_o (64 x 16),
// column j of Q_o holding right-hand side r_j of the 64 sources of the box at
// offset o from b_j (a zero column where b_j has no such neighbour, at the
// faces of the grid), so every column of an instruction shares the one G_o.
// Bound by the matrix cores.  It replaced a vector kernel (a wave per box, G
// from a table in LDS, one pass per right-hand side, bound by the LDS reads of
// G): 32^3 grid, 8 right-hand sides, FP64, forward and backward:
// 1109 to 136 us.
// v_mfma_f64_16x16x4f64, complex as three real products (one right-hand side)
// or four; lane l supplies
// A[l%16][l/16] and B[l/16][l%16], and accumulator register r of lane l holds
// row l/16 + 4 r (rows interleaved), column l%16.  A workgroup of 4 wavefronts
// owns a tile; wave w takes the offsets o = w, w + 4, ... for all 64 targets
// (four row tiles, 12 or 16 instructions per k-step of 4 sources) with a deep operand
// prefetch, and the four partial products are summed through LDS at the end.
// The workgroup first maps every (offset, box) to the first row of its sources
// -- the sorted rows of the neighbour box (gather) or its place in the target's
// segment (redundant) -- from the near lists of the tile's boxes, which are one
// contiguous run of the CSR.
constexpr int kColBoxes = kHelmColBoxes;
constexpr int kColWaves = 4;
static_assert(kColWaves == 4, "wave w finishes row tile w of the four");
// prefetch distances of the G and Q operands, in k-steps (the buffer rotation
// runs on across offsets of 16 k-steps each)
constexpr int kColPrefG = 3;
constexpr int kColPrefQ = 7;

// G blocks: double2 at [table][offset][source][target % 16][target / 16], the
// four row tiles of a target column next to each other, so a lane reads the
// four it needs in one 64-byte run; 64 zero entries follow (the sources of an
// absent neighbour).  A workgroup forms the 148 values G can take once.  The
// workgroups past the first g_wgs (all of them with a prepared plan) copy q
// into sorted order: one launch for what the product needs beforehand.
constexpr int kGreenEntries = 1024;
constexpr int kGreenWgs = 27 * 4096 / kGreenEntries;
template <class I>
__global__ __launch_bounds__(256) void k_prep64(const double *__restrict__ kh_dev, HelmInline inl,
                                                int32_t n_tables, double2 *__restrict__ out, int32_t g_wgs,
                                                const double2 *__restrict__ q, const int32_t *__restrict__ perm,
                                                I units, I nrhs, double2 *__restrict__ sorted) {
    __shared__ double2 s_g[kDistances];
    if (static_cast<int32_t>(blockIdx.x) >= g_wgs) {
        permute_entries(q, perm, units, nrhs, sorted, static_cast<I>(blockIdx.x) - static_cast<I>(g_wgs));
        return;
    }
    constexpr int per = 27 * 4096, wgs = kGreenWgs;
    const int tab = static_cast<int>(blockIdx.x) / wgs, e0 = (static_cast<int>(blockIdx.x) % wgs) * kGreenEntries;
    if (threadIdx.x < kDistances) s_g[threadIdx.x] = green(table_kh(inl, kh_dev, tab), threadIdx.x);
    __syncthreads();
#pragma unroll
    for (int k = 0; k < kGreenEntries / 256; ++k) {
        const int e = e0 + 256 * k + static_cast<int>(threadIdx.x);      // [o][s][c][r], target 16 r + c
        const int o = e >> 12, s = (e >> 6) & 63, i = 16 * (e & 3) + ((e >> 2) & 15);
        out[static_cast<int64_t>(tab) * per + e] = s_g[near_distance(o, s, i)];
    }
    if (blockIdx.x == 0 && threadIdx.x < 64)
        out[static_cast<int64_t>(n_tables) * per + threadIdx.x] = make_double2(0.0, 0.0);
}

// A tile's 27 offsets may be shared by H = 2, 4 or 7 workgroups (as many as the
// card has CUs for; a wavefront then takes four, two or one of them instead of
// seven): wave w of part p takes offsets o = 4 p + w + 4 H idx, the slots past
// the 27 offsets reading zero rows.  With H > 1 each part stores its
// result in sorted order to parts[p][.] (coalesced), and k_join_parts adds
// the parts in order and scatters the sum to the caller's order (FP64 atomic
// additions at the scattered caller rows took 7 us more on a 48^3 grid).  A
// prepared call on a 32^3 grid, one right-hand side: 40 us with two workgroups
// a tile, 26 us with seven.
template <bool RED, bool CONJ, bool ONE, int H>
__global__ __launch_bounds__(64 * kColWaves) void k_helm_mfma_cols64(
    int key_bits, HelmTiles ht, HelmInline inl, int32_t nrhs, const int32_t *__restrict__ leaf_start,
    const uint64_t *__restrict__ leaf_key, const int32_t *__restrict__ perm,
    const int64_t *__restrict__ nbr_start, const int32_t *__restrict__ nbr_idx,
    const int64_t *__restrict__ red_start, const int64_t *__restrict__ red_row, const double2 *__restrict__ src,
    const double2 *__restrict__ blocks, const double2 *__restrict__ zeros, const int32_t *__restrict__ inst_table,
    const double *__restrict__ inst_h, double2 *__restrict__ u, double2 *__restrict__ parts, int64_t n) {
    typedef double f64x4 __attribute__((ext_vector_type(4)));
    constexpr int VW = kColWaves * H;              // waves sharing a tile's offsets
    constexpr int NSL = (27 + VW - 1) / VW;        // offset slots per wave
    __shared__ ColMap<kColBoxes> s_map;
    const ColMapView sm = s_map.view();
    __shared__ double s_red[kColWaves][4][2][4][64];
    const int tid = threadIdx.x, lane = tid & 63;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int32_t b = static_cast<int32_t>(blockIdx.x) / H, part = static_cast<int32_t>(blockIdx.x) % H;
    const ColTile ct = col_tile<kColBoxes>(inl, ht, nrhs, inst_table, nullptr, inst_h, ht.tile0 + b);
    const int32_t cnt = ct.cnt, tab = ct.tab;
    const double sc64 = ct.sc64;
    const int li = lane & 15, kq = lane >> 4;
    const ColLane cl = col_lane<ONE>(ct, nrhs, li);
    col_map<RED, 64 * kColWaves>(sm, key_bits, cl.A0, cl.boxes, leaf_start, leaf_key, nbr_start, nbr_idx, red_start,
                                 red_row);

    const double2 *__restrict__ gbase = blocks + static_cast<int64_t>(tab) * (27 * 4096);
    // lane (kq, li) reads, at k-step kk, G_o[source 4 kk + kq][targets li, 16 + li, 32 + li, 48 + li]
    // (one 64-byte run) and Q[source 4 kk + kq] of column li; the slots past the 27
    // offsets and absent neighbours read the zero rows
    const int goff = (kq * 16 + li) * 4;
    const int vw = part * kColWaves + w;
    auto ptrs = [&](int idx, const double2 *&Gs, const double2 *&Qp) {
        const int o = vw + VW * idx;
        const int64_t row = o < 27 ? sm.row[o * kColBoxes + cl.box] : int64_t(-1);
        Gs = gbase + (o < 27 ? o : 0) * 4096;
        if constexpr (ONE)
            Qp = (row >= 0 ? src + row : zeros) + kq;
        else
            Qp = row >= 0 ? src + (row + kq) * nrhs + cl.rhs : zeros;
    };
    int64_t dst[4] = {0, 0, 0, 0};
    // One right-hand side: three real products per complex one, pa = sum Re G Re Q,
    // pb = sum Im G Im Q, pc = sum (Re G +- Im G)(Re Q + Im Q), the sums formed per
    // k-step.  Several: four, pa and pc the real and the imaginary part: an
    // imaginary part formed as pc - pa - pb carries the rounding of the real one,
    // which a caller with real q and a small kh sees (kh 1e-4: 1.1e-12 of Im u,
    // 3e-16 by four), and spreads an infinity of one part to the other.  They
    // start anew at every offset and are added to sr and si behind it: a chain of
    // 128 terms instead of up to 896 (32^3 grid, 8 right-hand sides: 9.4e-16
    // without, 4.4e-16 with).
    constexpr int NB = ONE ? 4 : 1, NC = ONE ? 1 : 4;
    const f64x4 zero = f64x4{0.0, 0.0, 0.0, 0.0};
    f64x4 pa[4], pb[NB], pc[4], sr[NC], si[NC];
#pragma unroll
    for (int rt = 0; rt < 4; ++rt) {
        pa[rt] = pc[rt] = zero;
        pb[rt % NB] = sr[rt % NC] = si[rt % NC] = zero;
    }
    {
        const double2 *Gs[NSL], *Qs[NSL];
#pragma unroll
        for (int idx = 0; idx < NSL; ++idx) ptrs(idx, Gs[idx], Qs[idx]);
        constexpr int NS = NSL * 16;
        double2 gbuf[kColPrefG + 1][4], qbuf[kColPrefQ + 1];
        auto load_g = [&](int st) {
            const double2 *g = Gs[st / 16] + (st % 16) * 256 + goff;
            double2(&gv)[4] = gbuf[st % (kColPrefG + 1)];
#pragma unroll
            for (int rt = 0; rt < 4; ++rt) gv[rt] = g[rt];
        };
        const double2 *qp = nullptr;
        int64_t qs = 0;
        auto load_q = [&](int st) {
            if constexpr (ONE) {
                qbuf[st % (kColPrefQ + 1)] = Qs[st / 16][(st % 16) * 4];
            } else {
                if (st % 16 == 0) {
                    qp = Qs[st / 16];
                    qs = qp == zeros ? 0 : 4 * static_cast<int64_t>(nrhs);
                }
                qbuf[st % (kColPrefQ + 1)] = *qp;
                qp += qs;
            }
        };
#pragma unroll
        for (int st = 0; st < kColPrefG; ++st) load_g(st);
#pragma unroll
        for (int st = 0; st < kColPrefQ; ++st) load_q(st);
        // the rows of the four targets this lane stores at the end: caller-order
        // rows, or sorted rows of this workgroup's part
        if (li < cnt) {
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int32_t sr = sm.tstart[cl.box] + 16 * w + kq + 4 * r;
                dst[r] = H == 1 ? perm[sr] : sr;
                if constexpr (!ONE) dst[r] = dst[r] * nrhs + cl.rhs;
            }
        }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int idx = 0; idx < NSL; ++idx) {
#pragma unroll
            for (int kk = 0; kk < 16; ++kk) {
                const int st = idx * 16 + kk;
                if (st + kColPrefG < NS) load_g(st + kColPrefG);
                if (st + kColPrefQ < NS) load_q(st + kColPrefQ);
                __builtin_amdgcn_sched_barrier(0);
                const double2(&gv)[4] = gbuf[st % (kColPrefG + 1)];
                const double2 q = qbuf[st % (kColPrefQ + 1)];
                if constexpr (ONE) {
                    const double qs = q.x + q.y;
#pragma unroll
                    for (int rt = 0; rt < 4; ++rt) {
                        const double gs = CONJ ? gv[rt].x - gv[rt].y : gv[rt].x + gv[rt].y;
                        pa[rt] = __builtin_amdgcn_mfma_f64_16x16x4f64(gv[rt].x, q.x, pa[rt], 0, 0, 0);
                        pb[rt] = __builtin_amdgcn_mfma_f64_16x16x4f64(gv[rt].y, q.y, pb[rt], 0, 0, 0);
                        pc[rt] = __builtin_amdgcn_mfma_f64_16x16x4f64(gs, qs, pc[rt], 0, 0, 0);
                    }
                } else {
                    // Im G meets -Im q and Re q (G q), or Im q and -Re q (conj(G) q)
                    const double nr = CONJ ? q.y : -q.y, ni = CONJ ? -q.x : q.x;
#pragma unroll
                    for (int rt = 0; rt < 4; ++rt) {
                        pa[rt] = __builtin_amdgcn_mfma_f64_16x16x4f64(gv[rt].x, q.x, kk == 0 ? zero : pa[rt], 0, 0, 0);
                        pc[rt] = __builtin_amdgcn_mfma_f64_16x16x4f64(gv[rt].x, q.y, kk == 0 ? zero : pc[rt], 0, 0, 0);
                    }
#pragma unroll
                    for (int rt = 0; rt < 4; ++rt) {
                        pa[rt] = __builtin_amdgcn_mfma_f64_16x16x4f64(gv[rt].y, nr, pa[rt], 0, 0, 0);
                        pc[rt] = __builtin_amdgcn_mfma_f64_16x16x4f64(gv[rt].y, ni, pc[rt], 0, 0, 0);
                    }
                }
                __builtin_amdgcn_sched_barrier(0);
            }
            if constexpr (!ONE)
#pragma unroll
                for (int rt = 0; rt < 4; ++rt) {
                    sr[rt] += pa[rt];
                    si[rt] += pc[rt];
                }
        }
    }
    // Three products: U = G Q: Re = pa - pb, Im = pc - pa - pb; with CONJ (conj G):
    // Re = pa + pb, Im = pc - pa + pb.  Wave w finishes row tile w from the four
    // waves' partials, in wave order.
#pragma unroll
    for (int rt = 0; rt < 4; ++rt)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            if constexpr (ONE) {
                s_red[w][rt][0][r][lane] = CONJ ? pa[rt][r] + pb[rt][r] : pa[rt][r] - pb[rt][r];
                s_red[w][rt][1][r][lane] = CONJ ? pc[rt][r] - pa[rt][r] + pb[rt][r] : pc[rt][r] - pa[rt][r] - pb[rt][r];
            } else {
                s_red[w][rt][0][r][lane] = sr[rt][r];
                s_red[w][rt][1][r][lane] = si[rt][r];
            }
        }
    __syncthreads();
    if (li < cnt) {
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            double tr = s_red[0][w][0][r][lane], ti = s_red[0][w][1][r][lane];
#pragma unroll
            for (int q = 1; q < kColWaves; ++q) {
                tr += s_red[q][w][0][r][lane];
                ti += s_red[q][w][1][r][lane];
            }
            if constexpr (H == 1)
                u[dst[r]] = make_double2(tr * sc64, ti * sc64);
            else
                parts[part * n + dst[r]] = make_double2(tr * sc64, ti * sc64);
        }
    }
}

// u[perm[s]][r] = the sum of parts[p][s][r] over the `share` parts, in order, for
// every sorted row s and right-hand side r (m = rows times right-hand sides).
__global__ void k_join_parts(const double2 *__restrict__ parts, int32_t share, const int32_t *__restrict__ perm,
                             int64_t m, int32_t nrhs, double2 *__restrict__ u) {
    const int64_t i = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
    if (i >= m) return;
    double2 v = parts[i];
    for (int p = 1; p < share; ++p) {
        const double2 b = parts[p * m + i];
        v.x += b.x;
        v.y += b.y;
    }
    if (nrhs == 1) {
        u[perm[i]] = v;
    } else {
        const int64_t s = i / nrhs;
        u[static_cast<int64_t>(perm[s]) * nrhs + (i - s * nrhs)] = v;
    }
}

}  // namespace

template <bool R, bool C, bool O, int H>
static void launch_cols64(const HelmholtzMfmaArgs &a, const HelmTiles &ht, const HelmInline &inl, int32_t n_tiles,
                          hipStream_t s) {
    k_helm_mfma_cols64<R, C, O, H><<<static_cast<unsigned>(n_tiles) * H, 64 * kColWaves, 0, s>>>(
        a.key_bits, ht, inl, a.nrhs, a.leaf_start, a.leaf_key, a.perm, a.nbr_start, a.nbr_idx, a.red_start, a.red_row,
        reinterpret_cast<const double2 *>(a.src), reinterpret_cast<const double2 *>(a.blocks),
        reinterpret_cast<const double2 *>(a.zeros), a.inst_table, a.inst_h, reinterpret_cast<double2 *>(a.u), a.parts,
        a.n * a.nrhs);
}

template <bool R, bool C, bool O>
static void launch_cols(const HelmholtzMfmaArgs &a, const HelmTiles &ht, const HelmInline &inl, int32_t n_tiles,
                        int32_t share, hipStream_t s) {
    if (share == 7) launch_cols64<R, C, O, 7>(a, ht, inl, n_tiles, s);
    else if (share == 4) launch_cols64<R, C, O, 4>(a, ht, inl, n_tiles, s);
    else if (share == 2) launch_cols64<R, C, O, 2>(a, ht, inl, n_tiles, s);
    else launch_cols64<R, C, O, 1>(a, ht, inl, n_tiles, s);
}

template <bool R, bool C>
static void launch_cols(const HelmholtzMfmaArgs &a, const HelmTiles &ht, const HelmInline &inl, int32_t n_tiles,
                        int32_t share, hipStream_t s) {
    if (a.nrhs == 1) launch_cols<R, C, true>(a, ht, inl, n_tiles, share, s);
    else launch_cols<R, C, false>(a, ht, inl, n_tiles, share, s);
}

p2p_status launch_prep64(const double *d_kh, const HelmInline &inl, int32_t n_tables, void *blocks, const void *q,
                         const int32_t *perm, int64_t n, int32_t nrhs, void *sorted, hipStream_t s) {
    const int64_t g_wgs = static_cast<int64_t>(n_tables) * kGreenWgs;
    const uint64_t units = sorted ? static_cast<uint64_t>(n) * static_cast<uint64_t>(nrhs) : 0;
    const int64_t wgs = g_wgs + static_cast<int64_t>((units + kPermuteEntries - 1) / kPermuteEntries);
    if (wgs == 0) return P2P_OK;
#define P2P_PREP64(I)                                                                                             \
    k_prep64<I><<<static_cast<unsigned>(wgs), 256, 0, s>>>(                                                       \
        d_kh, inl, n_tables, static_cast<double2 *>(blocks), static_cast<int32_t>(g_wgs),                         \
        static_cast<const double2 *>(q), perm, static_cast<I>(units), static_cast<I>(nrhs),                       \
        static_cast<double2 *>(sorted))
    // 32-bit entry indices while they fit (with room for the last workgroup's overshoot)
    if (units + kPermuteEntries < (uint64_t(1) << 32)) P2P_PREP64(uint32_t); else P2P_PREP64(uint64_t);
#undef P2P_PREP64
    P2P_LAUNCH_CHECK();
    return P2P_OK;
}

p2p_status launch_helmholtz_cols64(const HelmholtzMfmaArgs &a, const HelmTiles &ht, const HelmInline &inl,
                                   int32_t n_tiles, bool redundant, hipStream_t s) {
    if (n_tiles <= 0) return P2P_OK;
    int dev = 0, cus = 0;
    P2P_HIP(hipGetDevice(&dev));
    P2P_HIP(hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev));
    // as many workgroups per tile as still fit on the card's CUs
    const int32_t share = a.parts ? helm_cols64_share(n_tiles, cus) : 1;
    const bool cj = a.conj != 0;
    if (redundant) { if (cj) launch_cols<true, true>(a, ht, inl, n_tiles, share, s);
                     else launch_cols<true, false>(a, ht, inl, n_tiles, share, s); }
    else { if (cj) launch_cols<false, true>(a, ht, inl, n_tiles, share, s);
           else launch_cols<false, false>(a, ht, inl, n_tiles, share, s); }
    P2P_LAUNCH_CHECK();
    if (share > 1) {
        const int64_t m = a.n * a.nrhs;
        k_join_parts<<<grid_for(m, 256), 256, 0, s>>>(a.parts, share, a.perm, m, a.nrhs, reinterpret_cast<double2 *>(a.u));
        P2P_LAUNCH_CHECK();
    }
    return P2P_OK;
}

}  // namespace p2p
