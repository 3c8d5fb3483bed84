// Tree binning (Sec. 4: the stellar-dynamics tree is rebuilt every step):
// integer keys, and leaf boundaries over the sorted keys.
//
// Particles: c_d = floor(x_d 2^20), key = Morton(c).  The sort itself is
// radix_sort_pairs.  Leaves of an adaptive tree are found without walking
// the tree: over the sorted keys, let c[i] be the number of leading octal
// digits shared by keys i and i+1.  The node at level l that holds particle i
// contains exactly the run of neighbours reachable through pairs with
// c >= l, so its count is 1 + (run to the left) + (run to the right).  A
// particle's leaf is the shallowest node on its root path holding at most
// leaf_cap points (the split rule: split iff count > cap and level < depth),
// and that level is one more than the cap-th largest value of the merged,
// non-increasing sequences of running minima of c to the left and to the
// right of i.  A merge of leaf_cap steps finds it.
#include "p2p_internal.h"

namespace p2p {
namespace {

__global__ void k_particle_keys(const double *__restrict__ x, const double *__restrict__ y,
                                const double *__restrict__ z, int64_t n,
                                uint64_t *__restrict__ keys, int32_t *__restrict__ bad) {
    int64_t i = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const double p[3] = {x[i], y[i], z[i]};
    uint32_t c[3];
    bool ok = true;
#pragma unroll
    for (int d = 0; d < 3; ++d) {
        ok = ok && (p[d] >= 0.0 && p[d] < 1.0);
        // x * 2^20 is exact; truncation of a non-negative value is floor
        c[d] = ok ? static_cast<uint32_t>(p[d] * 1048576.0) : 0u;
    }
    // a point outside the domain: marked in its key for the sort by counting
    // (bad == null), else in the counts
    if (!ok && bad) atomicOr(bad, 1);
    keys[i] = ok || bad ? p2pd::morton3(c[0], c[1], c[2]) : kBadKey;
}

__global__ void k_grid_keys(const int32_t *__restrict__ n_side, const int64_t *__restrict__ off,
                            int32_t n_grids, int bits, int64_t n, uint64_t *__restrict__ keys) {
    int64_t p = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
    if (p >= n) return;
    // binary search of the instance: last g with off[g] <= p
    int lo = 0, hi = n_grids - 1;
    while (lo < hi) {
        int mid = (lo + hi + 1) >> 1;
        if (off[mid] <= p) lo = mid; else hi = mid - 1;
    }
    const int64_t ns = n_side[lo], loc = p - off[lo];
    const uint32_t i = static_cast<uint32_t>(loc % ns), j = static_cast<uint32_t>((loc / ns) % ns),
                   k = static_cast<uint32_t>(loc / (ns * ns));
    keys[p] = (static_cast<uint64_t>(lo) << (3 * bits)) | p2pd::morton3(i, j, k);
}

// Leading octal digits shared by two depth-20 keys (60-bit keys in 64-bit words).
__device__ inline int common_digits(uint64_t a, uint64_t b) {
    uint64_t x = a ^ b;
    return x == 0 ? 20 : (__clzll(static_cast<long long>(x)) - 4) / 3;
}

__global__ void k_pair_common(const uint64_t *__restrict__ sk, int64_t n, uint8_t *__restrict__ c,
                              const TreeCounts *__restrict__ tc) {
    if (tc->long_found != 0) return;
    int64_t i = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
    if (i + 1 < n) c[i] = static_cast<uint8_t>(common_digits(sk[i], sk[i + 1]));
}

// Ends every leaf-level kernel, called by all kMarkBlock threads of a workgroup:
// slot i's mark, and the workgroup's leaf starts and deepest level.
__device__ inline void leaf_mark(int64_t i, int64_t n, int l, bool first, uint8_t *__restrict__ mark,
                                 int32_t *__restrict__ leaf_counts) {
    __shared__ int s_cnt[kMarkBlock / 64], s_lev[kMarkBlock / 64];
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    if (i < n) mark[i] = static_cast<uint8_t>(l) | (first ? kLeafFirst : 0);
    const int cnt = __popcll(__ballot(i < n && first));
    int m = i < n ? l : 0;
    for (int o = 32; o > 0; o >>= 1) m = max(m, __shfl_xor(m, o, 64));
    if (lane == 0) {
        s_cnt[w] = cnt;
        s_lev[w] = m;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        int c = 0;
        for (int q = 0; q < kMarkBlock / 64; ++q) {
            c += s_cnt[q];
            m = max(m, s_lev[q]);
        }
        leaf_counts[blockIdx.x] = c | (m << kDeepShift);
    }
}

// Adaptive levels for any leaf_cap > 0.
__global__ void k_leaf_level_particles(const uint8_t *__restrict__ c, int64_t n, int depth,
                                       int leaf_cap, uint8_t *__restrict__ mark,
                                       int32_t *__restrict__ leaf_counts, const TreeCounts *__restrict__ tc) {
    if (tc->long_found != 0) return;
    const int64_t i = static_cast<int64_t>(blockIdx.x) * kMarkBlock + threadIdx.x;
    int l = depth;
    if (i < n) {
        // merge the running minima to the left (pairs i-1, i-2, ...) and to the
        // right (pairs i, i+1, ...); -1 marks an exhausted side
        int64_t left = i - 1, right = i;
        int mL = 127, mR = 127;
        int cl = (left >= 0) ? static_cast<int>(c[left]) : -1;
        int cr = (right < n - 1) ? static_cast<int>(c[right]) : -1;
        int v = -1;
        for (int t = 0; t < leaf_cap; ++t) {
            int candL = (left >= 0) ? min(mL, cl) : -1;
            int candR = (right < n - 1) ? min(mR, cr) : -1;
            if (candL < 0 && candR < 0) { v = -1; break; }
            if (candL >= candR) {
                v = candL; mL = candL; --left;
                cl = (left >= 0) ? static_cast<int>(c[left]) : -1;
            } else {
                v = candR; mR = candR; ++right;
                cr = (right < n - 1) ? static_cast<int>(c[right]) : -1;
            }
        }
        l = min(depth, v + 1);
    }
    // a new leaf starts at i unless slot i-1 shares i's level-l node
    leaf_mark(i, n, l, i < n && (i == 0 || static_cast<int>(c[i - 1]) < l), mark, leaf_counts);
}

// The same leaf levels for leaf_cap <= 64 without the merge: slot i's leaf
// level is the coarsest level l whose node around i holds at most leaf_cap
// slots (the merge's last common-digit count v satisfies v + 1 = that level;
// past the node the merge only meets smaller counts), capped at depth.  The
// node at level l spans the run of counts >= l on either side of i, and no
// run longer than 64 matters, so a wave of 64 slots reads the counts of
// slots -64..127 around it as three ballots per level, and each lane measures
// its run with one leading- and one trailing-ones count.  Levels are tried
// from the root down until every lane has its answer.  leaf_cap == 0: the
// uniform tree, every leaf at `depth`.
__global__ __launch_bounds__(kMarkBlock) void k_leaf_level_ballot(const uint64_t *__restrict__ sk, int64_t n,
                                                                  int depth, int leaf_cap,
                                                                  uint8_t *__restrict__ mark,
                                                                  int32_t *__restrict__ leaf_counts,
                                                                  const TreeCounts *__restrict__ tc) {
    __shared__ int8_t cs[256 + 128];   // cs[k] = c[b - 64 + k], -1 past either end
    const int64_t b = static_cast<int64_t>(blockIdx.x) * 256;
    const int t = threadIdx.x, lane = t & 63, wv = t >> 6;
    const bool skip = tc->long_found != 0;   // read beside the keys
    for (int k = t; k < 256 + 128; k += 256) {
        const int64_t j = b - 64 + k;
        cs[k] = (j >= 0 && j + 1 < n) ? static_cast<int8_t>(common_digits(sk[j], sk[j + 1])) : int8_t(-1);
    }
    __syncthreads();
    if (skip) return;
    // this wave's window: c of slots (wave's first) - 64 + k, k < 192, in three registers
    const int c0 = cs[64 * wv + lane], c1 = cs[64 * wv + 64 + lane], c2 = cs[64 * wv + 128 + lane];
    const int sh = lane;   // the lane's own count c[i] sits at window bit 64 + lane
    int lev = -1;
    for (int l = 0; l <= 21 && leaf_cap > 0; ++l) {
        const uint64_t W0 = __ballot(c0 >= l), W1 = __ballot(c1 >= l), W2 = __ballot(c2 >= l);
        // right: window bits 64 + lane .. 127 + lane; left: bits lane .. 63 + lane (top bit: c[i - 1])
        const uint64_t R = sh == 0 ? W1 : (W1 >> sh) | (W2 << (64 - sh));
        const uint64_t Lw = sh == 0 ? W0 : (W0 >> sh) | (W1 << (64 - sh));
        const int right = R == ~0ull ? 64 : __builtin_ctzll(~R);
        const int left = Lw == ~0ull ? 64 : __builtin_clzll(~Lw);
        if (lev < 0 && left + right + 1 <= leaf_cap) lev = l;
        if (__ballot(lev < 0) == 0) break;
    }
    const int64_t i = b + 64 * wv + lane;
    const int l = leaf_cap > 0 ? min(depth, lev) : depth;
    leaf_mark(i, n, l, i == 0 || static_cast<int>(cs[64 * wv + 63 + lane]) < l, mark, leaf_counts);
}

// The same leaf levels for leaf_cap <= kTileCap, a block of 256 slots at a
// time: the block first forms the common-digit counts of its slots and of
// leaf_cap slots on either side (the farthest the merge can reach) from the
// sorted keys into LDS, -1 past either end of the sequence, so the merge loop
// reads LDS instead of issuing a scattered byte load per step.
constexpr int kTileCap = 2048;
constexpr int kTileSlots = kMarkBlock;
__global__ __launch_bounds__(kTileSlots) void k_leaf_level_tile(const uint64_t *__restrict__ sk, int64_t n,
                                                                  int depth, int leaf_cap,
                                                                  uint8_t *__restrict__ mark,
                                                                  int32_t *__restrict__ leaf_counts,
                                                                  const TreeCounts *__restrict__ tc) {
    extern __shared__ int8_t cs[];   // cs[k] = c[b - leaf_cap + k], k < kTileSlots + 2 leaf_cap
    const int64_t b = static_cast<int64_t>(blockIdx.x) * kTileSlots;
    const int t = threadIdx.x, w = kTileSlots + 2 * leaf_cap;
    if (tc->long_found != 0) return;
    for (int k = t; k < w; k += kTileSlots) {
        const int64_t j = b - leaf_cap + k;
        cs[k] = (j >= 0 && j + 1 < n) ? static_cast<int8_t>(common_digits(sk[j], sk[j + 1])) : int8_t(-1);
    }
    __syncthreads();
    const int64_t i = b + t;
    // left slot i - 1 - dl at cs[t + leaf_cap - 1 - dl], right slot i + dr at cs[t + leaf_cap + dr]
    int kl = t + leaf_cap - 1, kr = t + leaf_cap;
    int mL = 127, mR = 127, v = -1;
    int cl = cs[kl], cr = cs[kr];
    // after step + 1 < leaf_cap moves, kl >= t and kr < t + 2 leaf_cap: both in the tile
    for (int step = 0; step < leaf_cap; ++step) {
        const int candL = min(mL, cl), candR = min(mR, cr);
        if (candL < 0 && candR < 0) { v = -1; break; }
        const bool more = step + 1 < leaf_cap;
        if (candL >= candR) {
            v = candL; mL = candL; --kl;
            if (more) cl = cs[kl];
        } else {
            v = candR; mR = candR; ++kr;
            if (more) cr = cs[kr];
        }
    }
    const int l = min(depth, v + 1);
    leaf_mark(i, n, l, i == 0 || static_cast<int>(cs[t + leaf_cap - 1]) < l, mark, leaf_counts);
}

__global__ __launch_bounds__(kMarkBlock) void k_leaf_flag_grids(const uint64_t *__restrict__ sk, int64_t n,
                                                                uint8_t *__restrict__ mark, int box_level,
                                                                int32_t *__restrict__ leaf_counts,
                                                                const TreeCounts *__restrict__ tc) {
    if (tc->long_found != 0) return;
    const int64_t i = static_cast<int64_t>(blockIdx.x) * kMarkBlock + threadIdx.x;
    leaf_mark(i, n, box_level, i < n && (i == 0 || (sk[i] >> 6) != (sk[i - 1] >> 6)), mark, leaf_counts);
}

// The counts of more slots than k_leaf_write sums: prefix sums of the leaf
// starts in place, their total and the deepest level (one workgroup).
__global__ __launch_bounds__(1024) void k_leaf_scan(int32_t *__restrict__ leaf_counts, int64_t nb,
                                                    TreeCounts *__restrict__ tc) {
    __shared__ int s_w[16], s_m[16];
    const int t = threadIdx.x, lane = t & 63, w = t >> 6;
    int carry = 0, m = 0;
    for (int64_t c0 = 0; c0 < nb; c0 += 1024) {
        const int64_t q = c0 + t;
        const int c = q < nb ? leaf_counts[q] : 0, v = c & ((1 << kDeepShift) - 1);
        m = max(m, c >> kDeepShift);
        int inc = v;
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            const int y = __shfl_up(inc, o, 64);
            if (lane >= o) inc += y;
        }
        if (lane == 63) s_w[w] = inc;
        __syncthreads();
        int off = carry;
        for (int k = 0; k < 16; ++k) {
            if (k < w) off += s_w[k];
            carry += s_w[k];
        }
        if (q < nb) leaf_counts[q] = off + inc - v;
        __syncthreads();
    }
    for (int o = 32; o > 0; o >>= 1) m = max(m, __shfl_xor(m, o, 64));
    if (lane == 0) s_m[w] = m;
    __syncthreads();
    if (t == 0) {
        for (int k = 0; k < 16; ++k) m = max(m, s_m[k]);
        tc->max_level = m;
        leaf_counts[nb] = carry;
    }
}

// One workgroup per kLeafTile slots: the leaves that start before them are the
// sum of leaf_counts (SCANNED: its prefix, already formed), a block scan gives
// each thread's slots their leaf ids, and the same workgroup writes perm and
// its inverse for its slots.  It stands for a scan of flags, the leaf writes,
// their maximum and the permutation, launches that each re-read the slots.
constexpr int kWriteBlock = 1024;
constexpr int kWriteItems = 2;
constexpr int kLeafTile = kWriteBlock * kWriteItems;
template <bool SCANNED>
__global__ __launch_bounds__(kWriteBlock) void k_leaf_write(
    const uint64_t *__restrict__ sk, const int32_t *__restrict__ vals, const uint8_t *__restrict__ mark, int64_t n,
    int kind, LongRuns lr, int64_t cap_leaves, const int32_t *__restrict__ leaf_counts, int64_t nb,
    TreeCounts *__restrict__ tc,
    int32_t *__restrict__ leaf_start, uint64_t *__restrict__ leaf_key, int8_t *__restrict__ leaf_level,
    int32_t *__restrict__ perm, int32_t *__restrict__ iperm) {
    constexpr int W = kWriteBlock / 64;
    __shared__ int32_t s_w[4][W];
    const int t = threadIdx.x, lane = t & 63, w = t >> 6;
    if (tc->long_found != 0) {
        if (blockIdx.x != 0) return;
        int32_t r = 0, k = 0;
        for (int64_t q = t; q < run_blocks(n); q += kWriteBlock) {
            r += lr.runs[q];
            k += lr.slots[q];
        }
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) {
            r += __shfl_xor(r, o, 64);
            k += __shfl_xor(k, o, 64);
        }
        if (lane == 0) {
            s_w[0][w] = r;
            s_w[1][w] = k;
        }
        __syncthreads();
        if (t == 0) {
            for (int q = 1; q < W; ++q) {
                r += s_w[0][q];
                k += s_w[1][q];
            }
            tc->long_runs = r;
            tc->long_slots = k;
        }
        return;
    }
    const int64_t i0 = static_cast<int64_t>(blockIdx.x) * kLeafTile;
    const int64_t b = i0 / kMarkBlock;   // the first count of this workgroup's slots
    // this thread's slots are consecutive
    const int64_t it = i0 + t * kWriteItems;
    uint8_t mk[kWriteItems];
    int cnt = 0;
#pragma unroll
    for (int k = 0; k < kWriteItems; ++k) {
        mk[k] = it + k < n ? mark[it + k] : 0;
        cnt += mk[k] >> 7;
    }
    int32_t before = 0, total = 0, deep = 0;
    if (!SCANNED)
        for (int64_t q = t; q < nb; q += kWriteBlock) {
            const int32_t c = leaf_counts[q], v = c & ((1 << kDeepShift) - 1);
            deep = max(deep, c >> kDeepShift);
            total += v;
            if (q < b) before += v;
        }
    int inc = cnt;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const int y = __shfl_up(inc, o, 64);
        if (lane >= o) inc += y;
    }
    if (!SCANNED) {
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) {
            before += __shfl_xor(before, o, 64);
            total += __shfl_xor(total, o, 64);
            deep = max(deep, __shfl_xor(deep, o, 64));
        }
    }
    if (lane == 63) {
        s_w[0][w] = inc;
        s_w[1][w] = before;
        s_w[2][w] = total;
        s_w[3][w] = deep;
    }
    __syncthreads();
    int32_t id = inc - cnt, L = 0;
    for (int q = 0; q < W; ++q) {
        if (q < w) id += s_w[0][q];
        if (!SCANNED) {
            id += s_w[1][q];
            L += s_w[2][q];
            deep = max(deep, s_w[3][q]);
        }
    }
    if (SCANNED) {
        id += leaf_counts[b];
        L = leaf_counts[nb];
    }
    if (blockIdx.x == 0 && t == 0) {
        tc->n_leaves = L;
        if (!SCANNED) tc->max_level = deep;
    }
    if (tc->bad != 0 || L > cap_leaves) return;
    if (blockIdx.x == 0 && t == 0) leaf_start[L] = static_cast<int32_t>(n);
#pragma unroll
    for (int k = 0; k < kWriteItems; ++k)
        if (mk[k] & kLeafFirst) {
            const int l = mk[k] & (kLeafFirst - 1);
            leaf_start[id] = static_cast<int32_t>(it + k);
            leaf_level[id] = static_cast<int8_t>(l);
            const uint64_t low_bits = (kind == P2P_TREE_PARTICLES) ? 3ull * (20 - l) : 6ull;
            const uint64_t mask = (low_bits >= 64) ? 0ull : ~((1ull << low_bits) - 1ull);
            leaf_key[id] = sk[it + k] & mask;
            ++id;
        }
    const int64_t i1 = min(n, i0 + kLeafTile);
    for (int64_t i = i0 + t; i < i1; i += kWriteBlock) {
        const int32_t v = vals[i];
        perm[i] = v;
        iperm[v] = static_cast<int32_t>(i);
    }
}

}  // namespace

p2p_status launch_particle_keys(const double *x, const double *y, const double *z, int64_t n,
                                uint64_t *keys, int32_t *bad_flag, hipStream_t s) {
    if (n <= 0) return P2P_OK;
    k_particle_keys<<<grid_for(n, 256), 256, 0, s>>>(x, y, z, n, keys, bad_flag);
    P2P_LAUNCH_CHECK();
    return P2P_OK;
}

p2p_status launch_grid_keys(const int32_t *d_n_side, const int64_t *d_point_off, int32_t n_grids,
                            int bits, int64_t n, uint64_t *keys, hipStream_t s) {
    if (n <= 0) return P2P_OK;
    k_grid_keys<<<grid_for(n, 256), 256, 0, s>>>(d_n_side, d_point_off, n_grids, bits, n, keys);
    P2P_LAUNCH_CHECK();
    return P2P_OK;
}

p2p_status launch_leaf_levels(const uint64_t *skeys, int64_t n, int kind, int depth, int leaf_cap,
                              uint8_t *pair_common, uint8_t *mark, int32_t *leaf_counts, const TreeCounts *tc,
                              hipStream_t s) {
    if (n <= 0) return P2P_OK;
    const unsigned g = grid_for(n, kMarkBlock);
    if (kind == P2P_TREE_PARTICLES && leaf_cap <= 64) {
        k_leaf_level_ballot<<<g, kMarkBlock, 0, s>>>(skeys, n, depth, leaf_cap, mark, leaf_counts, tc);
    } else if (kind == P2P_TREE_PARTICLES && leaf_cap <= kTileCap) {
        k_leaf_level_tile<<<g, kMarkBlock, kTileSlots + 2 * leaf_cap, s>>>(skeys, n, depth, leaf_cap, mark,
                                                                           leaf_counts, tc);
    } else if (kind == P2P_TREE_PARTICLES) {
        if (n > 1) {
            k_pair_common<<<grid_for(n - 1, 256), 256, 0, s>>>(skeys, n, pair_common, tc);
            P2P_LAUNCH_CHECK();
        }
        k_leaf_level_particles<<<g, kMarkBlock, 0, s>>>(pair_common, n, depth, leaf_cap, mark, leaf_counts, tc);
    } else {
        k_leaf_flag_grids<<<g, kMarkBlock, 0, s>>>(skeys, n, mark, depth, leaf_counts, tc);
    }
    P2P_LAUNCH_CHECK();
    return P2P_OK;
}

p2p_status launch_leaf_write(const uint64_t *skeys, const int32_t *vals, const uint8_t *mark, int64_t n, int kind,
                             const LongRuns &lr, int64_t cap_leaves, int32_t *leaf_counts, TreeCounts *tc, int32_t *leaf_start,
                             uint64_t *leaf_key, int8_t *leaf_level, int32_t *perm, int32_t *iperm, hipStream_t s) {
    if (n <= 0) return P2P_OK;
    // beyond this many counts (4M slots) their sum in every workgroup costs more than one launch that scans them
    constexpr int64_t kSumCounts = 16384;
    const int64_t nb = leaf_count_elems(n);
    const unsigned g = grid_for(n, kLeafTile);
    if (nb <= kSumCounts) {
        k_leaf_write<false><<<g, kWriteBlock, 0, s>>>(skeys, vals, mark, n, kind, lr, cap_leaves, leaf_counts, nb, tc,
                                                      leaf_start, leaf_key, leaf_level, perm, iperm);
    } else {
        k_leaf_scan<<<1, 1024, 0, s>>>(leaf_counts, nb, tc);
        P2P_LAUNCH_CHECK();
        k_leaf_write<true><<<g, kWriteBlock, 0, s>>>(skeys, vals, mark, n, kind, lr, cap_leaves, leaf_counts, nb, tc,
                                                     leaf_start, leaf_key, leaf_level, perm, iperm);
    }
    P2P_LAUNCH_CHECK();
    return P2P_OK;
}

}  // namespace p2p
