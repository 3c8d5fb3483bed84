// Near-field lists (the E2 neighbourhood, Sec. 5.1): for every leaf A, every leaf B whose closed cube
// touches A's, A included, in ascending leaf id.
//
// A leaf touching A either covers one of the 27 cells of A's size around A (A
// itself in the middle) or lies inside one.  One lane per cell finds, by binary
// search over the sorted leaf keys, the contiguous range of leaves that meet
// its cell.  The ranges of different cells are disjoint, except that one large
// leaf may cover several cells; those duplicates are dropped and the ranges are
// put in key order, which is leaf-id order.  The candidates are then tested in
// parallel, 64 per step, and the adjacent ones written with a ballot prefix, so
// the list comes out ascending.  Where there are many, the cell that encloses
// 64 successive candidates is tested first, one such chunk per lane, and only
// the chunks whose cell touches A are read.
//
// The first pass takes successive leaves of one size and one parent together,
// up to 8 to a wavefront: their cells are the 64 of the 4^3 block around the
// parent, one per lane, and every candidate is read once and tested against
// each of them.  A candidate that reaches a leaf only through another's cell
// does not touch it, so the lists are the same.
//
// The counting pass also sums, per leaf A, the points of the
// leaves in nbr(A): the length of A's segment in the redundant layout.
//
// The searches start from a directory over the top bits of the key: dir[p]
// is the first leaf whose key is at least p << shift, so a key's bucket bounds
// its search to the leaves of that bucket.
//
// Periodic lists (particles on the unit torus): a cell past a face of the
// domain wraps to the opposite side and carries the image code of that wrap,
// c = (sx+1) + 3 (sy+1) + 9 (sz+1); its leaves are tested shifted by
// (sx, sy, sz) domain edges.  Ranges are deduplicated and ordered by (c, lo),
// so the list comes out ascending in (c, B); one leaf may appear under
// several codes.
#include "p2p_internal.h"

namespace p2p {
namespace {

constexpr int kNbrWaves = 4;
constexpr int kNbrSlots = kNbrSlotsPerLeaf;

// First index in [lo, hi) with a[i] >= v.
__device__ inline int64_t bound_in(const uint64_t *__restrict__ a, int64_t lo, int64_t hi, uint64_t v) {
    while (lo < hi) {
        const int64_t mid = (lo + hi) >> 1;
        if (a[mid] < v) lo = mid + 1; else hi = mid;
    }
    return lo;
}

// Also clears the two counters of the counting pass that follows (lists over
// kNbrSlots entries, heavy leaves).
__global__ void k_key_directory(const uint64_t *__restrict__ leaf_key, int64_t L, int dir_bits,
                                int shift, int32_t *__restrict__ dir, int32_t *__restrict__ counters) {
    const int64_t p = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
    const int64_t nb = (int64_t(1) << dir_bits) + 1;
    if (p == 0) {
        counters[0] = 0;
        counters[1] = 0;
    }
    if (p >= nb) return;
    dir[p] = (p == nb - 1) ? static_cast<int32_t>(L)
                           : static_cast<int32_t>(bound_in(leaf_key, 0, L, static_cast<uint64_t>(p) << shift));
}

__device__ inline void wave_sync() {
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

// Count: counts[A], segs[A] and the first kNbrSlots entries of nbr(A) into
// slots[A * kNbrSlots ...]; a longer list is appended to the end of heavy[].
// Fill: those lists into nbr_idx[nbr_start[A] ...].
enum { kNbrCount = 0, kNbrFill = 1 };

// A leaf with more candidates than this (a large leaf beside a finely split
// region) is left to k_neighbors_heavy, which spreads its candidates over a
// whole workgroup; in one wavefront it would set the time of the whole pass.
// 700,001 periodic points, 512: 43 us and 39 us for the heavy leaves of both
// passes; 256: 41 and 52.
constexpr int32_t kHeavyCands = 512;
constexpr int kHeavyWaves = 16;
constexpr unsigned kHeavyGrid = 512;
constexpr unsigned kFillGrid = 1024;
constexpr int kChunk = 64;          // candidates tested in one step
constexpr int kSegChunks = 4096;    // chunks a heavy leaf's workgroup holds at a time

// What one leaf's search needs: the candidate (source) tree's arrays and key
// directory, the target leaves' keys and levels (the same tree for plain
// lists, another one for remote lists), and the key layout.
struct NbrTree {
    const uint64_t *leaf_key;
    const int8_t *leaf_level;
    const int32_t *leaf_start;
    const int32_t *dir;
    int64_t L;
    const uint64_t *tkey;
    const int8_t *tlevel;
    int64_t Lt;
    int key_bits, inst_shift, dir_bits, dir_shift;
};

// Leaf A's geometry in key units: anchor a, edge sA.
struct NbrLeaf {
    int32_t a[3];
    int32_t sA, dim;
    uint64_t local_mask, inst_bits;
    int lA;
};

__device__ inline NbrLeaf nbr_leaf(const NbrTree &t, int64_t A) {
    NbrLeaf f;
    const uint64_t kA = t.tkey[A];
    f.lA = t.tlevel[A];
    f.dim = int32_t(1) << t.key_bits;   // key_bits <= 20
    f.sA = int32_t(1) << (t.key_bits - f.lA);
    f.local_mask = (3 * t.key_bits >= 64) ? ~0ull : ((1ull << (3 * t.key_bits)) - 1ull);
    f.inst_bits = (t.inst_shift >= 64) ? 0ull : (kA >> t.inst_shift) << t.inst_shift;
    const uint64_t local = kA & f.local_mask;
    f.a[0] = static_cast<int32_t>(p2pd::compact3(local));
    f.a[1] = static_cast<int32_t>(p2pd::compact3(local >> 1));
    f.a[2] = static_cast<int32_t>(p2pd::compact3(local >> 2));
    return f;
}

// Candidate ranges in (code, lo) order, range r held by lane r: its first leaf,
// the candidates of the ranges before it, its image code (PER).
struct NbrRanges {
    int32_t lo, pre, code;
    int32_t total;   // candidates, the same in every lane
};

// The leaves [lo, hi) that meet the cell at c (may lie past the domain's faces
// by one cell) of the size of leaf f.  False if there is none; with PER the
// cell wraps, and its image code goes to `code`.
template <bool PER>
__device__ inline bool cell_range(const NbrTree &t, const NbrLeaf &f, int32_t (&c)[3], int32_t &lo, int32_t &hi,
                                  int &code) {
    const int32_t dim = f.dim;
    if constexpr (PER) {
        // c lies in [-sA, dim + sA) with sA <= dim: one wrap per axis
        int wrap[3];
#pragma unroll
        for (int d = 0; d < 3; ++d) {
            wrap[d] = c[d] < 0 ? -1 : (c[d] >= dim ? 1 : 0);
            c[d] -= wrap[d] * dim;
        }
        code = (wrap[0] + 1) + 3 * (wrap[1] + 1) + 9 * (wrap[2] + 1);
    } else if (c[0] < 0 || c[1] < 0 || c[2] < 0 || c[0] >= dim || c[1] >= dim || c[2] >= dim) {
        return false;
    }
    const uint64_t kC = f.inst_bits | p2pd::morton3(static_cast<uint32_t>(c[0]), static_cast<uint32_t>(c[1]),
                                                    static_cast<uint32_t>(c[2]));
    // both ends of the cell, searched together: first leaf past kC, first leaf past the cell
    const uint64_t kE = kC + (1ull << (3 * (t.key_bits - f.lA))), top = 1ull << t.dir_bits;
    const uint64_t p0 = kC >> t.dir_shift, p1 = kE >> t.dir_shift;
    int32_t l0 = t.dir[min(p0, top)], h0 = t.dir[min(p0 + 1, top)];
    int32_t l1 = t.dir[min(p1, top)], h1 = t.dir[min(p1 + 1, top)];
    while (l0 < h0 || l1 < h1) {
        const int32_t m0 = (l0 + h0) >> 1, m1 = (l1 + h1) >> 1;
        const bool go0 = l0 < h0, go1 = l1 < h1;
        const uint64_t v0 = go0 ? t.leaf_key[m0] : 0ull, v1 = go1 ? t.leaf_key[m1] : 0ull;
        if (go0) {
            if (v0 <= kC) l0 = m0 + 1; else h0 = m0;
        }
        if (go1) {
            if (v1 < kE) l1 = m1 + 1; else h1 = m1;
        }
    }
    const int32_t j = l0 - 1;
    bool covers = false;
    int lj = 0;
    if (j >= 0) {
        lj = t.leaf_level[j];
        covers = kC < t.leaf_key[j] + (1ull << (3 * (t.key_bits - lj)));   // leaf_key[j] <= kC by construction
    }
    lo = covers ? j : j + 1;
    // a covering leaf at least as large as the cell holds all of it (aligned cubes)
    hi = covers && lj <= f.lA ? j + 1 : l1;
    return lo < hi;
}

// Called by one whole wavefront: the ranges [lo, hi) of the first N lanes in
// (code, lo) order.  Ranges are disjoint or the same (one large leaf covering
// several cells of one image), so with the sorted ones side by side a duplicate
// is dropped and successive ranges are joined.  s: 3 x 64 words of LDS, this
// wavefront's own.  The values that every lane compares come by readlane: as
// shuffles they cost their LDS latency one after the other, more than the
// searches.
template <int N, bool PER>
__device__ NbrRanges order_ranges(bool valid, int32_t lo, int32_t hi, int code, int32_t (&s)[3][64]) {
    const int lane = threadIdx.x & 63;
    if (!valid) lo = INT32_MAX;   // behind every leaf
    if (PER && !valid) code = 27;
    int rank = 0;
#pragma unroll
    for (int q = 0; q < N; ++q) {
        const int32_t loq = __builtin_amdgcn_readlane(lo, q);
        bool less = loq < lo || (loq == lo && q < lane);
        if constexpr (PER) {
            const int cq = __builtin_amdgcn_readlane(code, q);
            less = cq < code || (cq == code && less);
        }
        rank += less ? 1 : 0;
    }
    const int nv = __popcll(__ballot(valid));
    if (valid) {
        s[0][rank] = lo;
        s[1][rank] = hi;
        if constexpr (PER) s[2][rank] = code;
    }
    wave_sync();
    const bool has = lane < nv;
    lo = has ? s[0][lane] : INT32_MAX;
    hi = has ? s[1][lane] : 0;
    code = PER && has ? s[2][lane] : 13;
    const int32_t hi_prev = __shfl_up(hi, 1, 64);
    const int code_prev = PER ? __shfl_up(code, 1, 64) : 13;
    const bool head = has && (lane == 0 || lo > hi_prev || code != code_prev);
    const uint64_t heads = __ballot(head);
    const uint64_t after = lane == 63 ? 0ull : heads >> (lane + 1);
    const bool tail = has && (lane + 1 == nv || (after & 1));
    const int at = __popcll(heads & (lane == 63 ? ~0ull : (2ull << lane) - 1)) - 1;
    wave_sync();
    if (head) {
        s[0][at] = lo;
        if constexpr (PER) s[2][at] = code;
    }
    if (tail) s[1][at] = hi;
    wave_sync();
    NbrRanges r;
    const bool in = lane < __popcll(heads);
    r.lo = in ? s[0][lane] : 0;
    r.code = PER && in ? s[2][lane] : 13;
    const int32_t len = in ? s[1][lane] - r.lo : 0;
    int32_t inc = len;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const int32_t y = __shfl_up(inc, o, 64);
        if (lane >= o) inc += y;
    }
    r.total = __builtin_amdgcn_readlane(inc, 63);
    r.pre = in ? inc - len : INT32_MAX;
    wave_sync();   // the LDS words may be rewritten
    return r;
}

// The candidate ranges of one leaf, called by one whole wavefront.
template <bool PER>
__device__ NbrRanges nbr_ranges(const NbrTree &t, const NbrLeaf &f, int32_t (&s)[3][64]) {
    const int lane = threadIdx.x & 63;
    int32_t lo = 0, hi = 0;
    int code = 13;
    bool valid = false;
    if (lane < 27) {
        int32_t c[3] = {f.a[0] + (lane % 3 - 1) * f.sA, f.a[1] + ((lane / 3) % 3 - 1) * f.sA,
                        f.a[2] + (lane / 9 - 1) * f.sA};
        valid = cell_range<PER>(t, f, c, lo, hi, code);
    }
    return order_ranges<27, PER>(valid, lo, hi, code, s);
}

// Where candidate cidx (< total) lies: leaf cidx + off, image code `code`.
// Called by whole wavefronts, cidx any value >= 0.
template <bool PER>
__device__ inline void nbr_place(const NbrRanges &r, int32_t cidx, int32_t &off, int &code) {
    int q = 0;   // last range with pre <= cidx
#pragma unroll
    for (int step = 32; step > 0; step >>= 1)
        if (__shfl(r.pre, q + step, 64) <= cidx) q += step;
    off = __shfl(r.lo - r.pre, q, 64);
    code = PER ? __shfl(r.code, q, 64) : 13;
}

// The same for the chunk of candidates c0 + lane: the ranges that begin in the
// chunk mark their place in 64 words of LDS, and a lane's range is the count of
// the places up to its own.
template <bool PER>
__device__ inline void chunk_place(const NbrRanges &r, int32_t c0, int32_t (&s)[64], int32_t &off, int &code) {
    const int lane = threadIdx.x & 63;
    s[lane] = 0;
    wave_sync();
    if (r.pre > c0 && r.pre - c0 < kChunk) s[r.pre - c0] = 1;
    wave_sync();
    const uint64_t begins = __ballot(s[lane] != 0);
    wave_sync();
    const int q = __popcll(__ballot(r.pre <= c0)) - 1 + __popcll(begins & (lane == 63 ? ~0ull : (2ull << lane) - 1));
    off = __shfl(r.lo - r.pre, q, 64);
    code = PER ? __shfl(r.code, q, 64) : 13;
}

// The corner of a cube by its key, moved to image `code`.
template <bool PER>
__device__ inline void corner(const NbrLeaf &f, uint64_t key, int code, int32_t (&b)[3]) {
    b[0] = static_cast<int32_t>(p2pd::compact3(key));
    b[1] = static_cast<int32_t>(p2pd::compact3(key >> 1));
    b[2] = static_cast<int32_t>(p2pd::compact3(key >> 2));
    if constexpr (PER) {
        b[0] += (code % 3 - 1) * f.dim;
        b[1] += ((code / 3) % 3 - 1) * f.dim;
        b[2] += (code / 9 - 1) * f.dim;
    }
}

// Candidate `lane` of chunk ch: leaf B, image code cB, and whether there is one
// and it touches A.
template <bool PER>
__device__ inline bool nbr_candidate(const NbrTree &t, const NbrLeaf &f, const NbrRanges &r, int32_t ch,
                                     int32_t (&s_mark)[64], int32_t &B, int &cB) {
    const int32_t cidx = ch * kChunk + static_cast<int32_t>(threadIdx.x & 63);
    int32_t off;
    chunk_place<PER>(r, ch * kChunk, s_mark, off, cB);
    if (cidx >= r.total) return false;
    B = cidx + off;
    const int32_t s = int32_t(1) << (t.key_bits - t.leaf_level[B]);
    int32_t b[3];
    corner<PER>(f, t.leaf_key[B] & f.local_mask, cB, b);
    bool adj = true;
#pragma unroll
    for (int d = 0; d < 3; ++d) adj = adj && f.a[d] <= b[d] + s && b[d] <= f.a[d] + f.sA;
    return adj;
}

// Whether chunk ch of the candidates may hold one that touches the cube at f.a
// of edge `edge`: false if the chunk lies in one run of successive leaves and
// the smallest cell around its first and last leaf does not touch the cube.
// All of a chunk's leaves lie inside that cell: they are disjoint aligned cubes
// between two whose corners it holds.  Called by whole wavefronts, ch any value.
template <bool PER>
__device__ inline bool chunk_near(const NbrTree &t, const NbrLeaf &f, int32_t edge, const NbrRanges &r, int32_t ch) {
    const int64_t c0 = static_cast<int64_t>(ch) * kChunk;
    const bool in = c0 < r.total;
    const int32_t i0 = in ? static_cast<int32_t>(c0) : 0;
    const int32_t i1 = in ? min(r.total, i0 + kChunk) - 1 : 0;
    int32_t o0, o1;
    int code0, code1;
    nbr_place<PER>(r, i0, o0, code0);
    nbr_place<PER>(r, i1, o1, code1);
    if (!in) return false;
    if (o0 != o1 || code0 != code1 || i0 == i1) return true;
    const uint64_t k0 = t.leaf_key[i0 + o0] & f.local_mask, k1 = t.leaf_key[i1 + o1] & f.local_mask;
    const int m = (64 - __clzll(static_cast<long long>(k0 ^ k1)) + 2) / 3;
    int32_t b[3];
    corner<PER>(f, (k0 >> (3 * m)) << (3 * m), code0, b);
    bool near = true;
#pragma unroll
    for (int d = 0; d < 3; ++d) near = near && f.a[d] <= b[d] + (int32_t(1) << m) && b[d] <= f.a[d] + edge;
    return near;
}

// The counting pass: one wavefront per run of successive leaves of one size and
// one parent, found from the keys beside them; the wavefronts of the other
// leaves of a run have nothing to do.  Runs with more than kHeavyCands
// candidates go to k_neighbors_heavy leaf by leaf, at the front of heavy[].
// Bound by the latency of a wavefront's chain (searches, ordering, chunks) and
// by the lines that the searches touch, one per lane and step, so what counts
// is how few searches there are and how short the chain is.  2^21 clustered
// points: a wavefront per leaf took 231 us, 192 us with both ends of a cell
// searched together and the ranges compared by readlane, 128 us with the leaves
// of a parent taken together, 73 us with successive ranges joined and a
// candidate's range found by marks instead of a loop over the ranges.
template <bool PER>
__global__ __launch_bounds__(64 * kNbrWaves) void k_neighbors_count(
    NbrTree t, int32_t *__restrict__ counts, int32_t *__restrict__ segs, int32_t *__restrict__ slots,
    int8_t *__restrict__ slot_code, int32_t *__restrict__ counters, int32_t *__restrict__ heavy) {
    __shared__ int32_t s_w[kNbrWaves][3][64];
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const uint64_t below = (lane == 0) ? 0ull : (~0ull >> (64 - lane));
    const int64_t A = static_cast<int64_t>(blockIdx.x) * kNbrWaves + w;
    if (A >= t.Lt) return;
    // ---- the run: lane i holds leaf A - 1 + i
    const int64_t i = A - 1 + lane;
    uint64_t ki = 0;
    int li = -1;
    if (lane < 9 && i >= 0 && i < t.Lt) {
        ki = t.tkey[i];
        li = t.tlevel[i];
    }
    const uint64_t kA = __shfl(ki, 1, 64);
    const int lA = __builtin_amdgcn_readlane(li, 1);
    // key bits below the parent's; a root has no parent (the next bits may number grid instances)
    const int up = 3 * (t.key_bits - lA) + 3;
    const bool same = lA > 0 ? li == lA && (ki >> up) == (kA >> up) : lane == 1;
    const uint32_t run = static_cast<uint32_t>(__ballot(same)) & 0x1ff;
    if (run & 1) return;                                       // leaf A - 1 leads it
    const int members = __builtin_ctz(~(run >> 1));            // leaves A .. A + members - 1
    // their octants of the parent, and the parent's block of cells
    const int oct = lA > 0 ? static_cast<int>(ki >> (up - 3)) & 7 : 0;
    uint32_t present = 0;
#pragma unroll
    for (int q = 0; q < 8; ++q)
        if (q < members) present |= 1u << __builtin_amdgcn_readlane(oct, q + 1);
    NbrLeaf f = nbr_leaf(t, A);
    const int32_t sA = f.sA;
#pragma unroll
    for (int d = 0; d < 3; ++d) f.a[d] &= ~(2 * sA - 1);
    const int cx = (lane & 3) - 1, cy = ((lane >> 2) & 3) - 1, cz = (lane >> 4) - 1;
    const uint32_t reach = (cx < 0 ? 0x55u : cx > 1 ? 0xaau : 0xffu) & (cy < 0 ? 0x33u : cy > 1 ? 0xccu : 0xffu) &
                           (cz < 0 ? 0x0fu : cz > 1 ? 0xf0u : 0xffu);   // octants this cell is beside
    int32_t lo = 0, hi = 0;
    int code = 13;
    bool valid = false;
    if (reach & present) {
        int32_t c[3] = {f.a[0] + cx * sA, f.a[1] + cy * sA, f.a[2] + cz * sA};
        valid = cell_range<PER>(t, f, c, lo, hi, code);
    }
    const NbrRanges r = order_ranges<64, PER>(valid, lo, hi, code, s_w[w]);
    if (r.total > kHeavyCands) {
        int32_t at = 0;
        if (lane == 0) at = atomicAdd(&counters[1], members);
        at = __builtin_amdgcn_readfirstlane(at);
        if (lane < members) heavy[at + lane] = static_cast<int32_t>(A + lane);
        return;
    }
    // ---- test candidates, 64 at a time, in ascending (code, leaf id)
    const int32_t nch = (r.total + kChunk - 1) / kChunk;   // at most kHeavyCands / kChunk
    uint64_t todo = nch > 3 ? __ballot(chunk_near<PER>(t, f, 2 * sA, r, lane)) : (1ull << nch) - 1;
    int32_t written[8], occ[8];   // per octant: entries (the same in every lane), points of this lane's entries
#pragma unroll
    for (int q = 0; q < 8; ++q) written[q] = occ[q] = 0;
    while (todo != 0) {
        const int32_t c0 = __builtin_ctzll(todo) * kChunk, cidx = c0 + lane;
        todo &= todo - 1;
        int32_t off;
        int cB;
        chunk_place<PER>(r, c0, s_w[w][0], off, cB);
        const bool in = cidx < r.total;
        const int32_t B = in ? cidx + off : 0;
        const int32_t s = int32_t(1) << (t.key_bits - t.leaf_level[B]);
        const int32_t pts = t.leaf_start[B + 1] - t.leaf_start[B];
        int32_t b[3];
        corner<PER>(f, t.leaf_key[B] & f.local_mask, cB, b);
        bool ok[3][2];
#pragma unroll
        for (int d = 0; d < 3; ++d)
#pragma unroll
            for (int h = 0; h < 2; ++h)
                ok[d][h] = in && f.a[d] + h * sA <= b[d] + s && b[d] <= f.a[d] + (h + 1) * sA;
        int32_t m = 0;
#pragma unroll
        for (int q = 0; q < 8; ++q) {
            if (!((present >> q) & 1)) continue;
            const bool adj = ok[0][q & 1] && ok[1][(q >> 1) & 1] && ok[2][q >> 2];
            const uint64_t bal = __ballot(adj);
            const int32_t pos = written[q] + __popcll(bal & below);
            if (adj) {
                occ[q] += pts;
                if (pos < kNbrSlots) {
                    slots[(A + m) * kNbrSlots + pos] = B;
                    if constexpr (PER) slot_code[(A + m) * kNbrSlots + pos] = static_cast<int8_t>(cB);
                }
            }
            written[q] += __popcll(bal);
            ++m;
        }
    }
    int32_t m = 0;
#pragma unroll
    for (int q = 0; q < 8; ++q) {
        if (!((present >> q) & 1)) continue;
        int32_t sum = occ[q];
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) sum += __shfl_xor(sum, o, 64);
        if (lane == 0) {
            counts[A + m] = written[q];
            segs[A + m] = sum;
            if (written[q] > kNbrSlots) heavy[t.Lt - 1 - atomicAdd(&counters[0], 1)] = static_cast<int32_t>(A + m);
        }
        ++m;
    }
}

// The lists over kNbrSlots entries, one wavefront each, by workgroup b of nb.
template <bool PER>
__device__ inline void fill_long_lists(const NbrTree &t, uint32_t b, uint32_t nb, const int32_t *__restrict__ counters,
                                       const int32_t *__restrict__ heavy, const int64_t *__restrict__ nbr_start,
                                       int32_t *__restrict__ nbr_idx, int8_t *__restrict__ nbr_shift) {
    __shared__ int32_t s_w[kNbrWaves][3][64];
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const uint64_t below = (lane == 0) ? 0ull : (~0ull >> (64 - lane));
    const int64_t work = counters[0];
    for (int64_t h = static_cast<int64_t>(b) * kNbrWaves + w; h < work; h += static_cast<int64_t>(nb) * kNbrWaves) {
        const int64_t A = heavy[t.Lt - 1 - h];
        const NbrLeaf f = nbr_leaf(t, A);
        const NbrRanges r = nbr_ranges<PER>(t, f, s_w[w]);
        const int32_t nch = (r.total + kChunk - 1) / kChunk;   // at most kHeavyCands / kChunk
        uint64_t todo = nch > 2 ? __ballot(chunk_near<PER>(t, f, f.sA, r, lane)) : (1ull << nch) - 1;
        int64_t out = nbr_start[A];
        while (todo != 0) {
            const int32_t ch = __builtin_ctzll(todo);
            todo &= todo - 1;
            int32_t B = 0;
            int cB = 13;
            const bool adj = nbr_candidate<PER>(t, f, r, ch, s_w[w][0], B, cB);
            const uint64_t bal = __ballot(adj);
            if (adj) {
                const int64_t p = out + __popcll(bal & below);
                nbr_idx[p] = B;
                if constexpr (PER) nbr_shift[p] = static_cast<int8_t>(cB);
            }
            out += __popcll(bal);
        }
    }
}

// The leaves heavy[0 .. counters[1]), one workgroup each (grid-stride).  The
// first wavefront finds the ranges; the chunks of candidates that may touch A
// are listed in order, kSegChunks at a time, and shared out evenly; each
// chunk's adjacent candidates are kept as a mask, whose counts give every
// wavefront its first list position, and FILL writes the entries from the
// masks.  What it costs follows the surface of A, not the volume around it:
// 700,001 periodic points 19 us counting and 20 us filling (113 and 80 us with
// every candidate tested twice).
template <int MODE, bool PER>
__global__ __launch_bounds__(64 * kHeavyWaves) void k_neighbors_heavy(
    NbrTree t, int32_t *__restrict__ counts, int32_t *__restrict__ segs, const int32_t *__restrict__ counters,
    const int32_t *__restrict__ heavy, const int64_t *__restrict__ totals, int64_t cap,
    const int64_t *__restrict__ nbr_start, int32_t *__restrict__ nbr_idx, int8_t *__restrict__ nbr_shift) {
    __shared__ int32_t s_r[3][64];                // the ranges: first leaf, prefix, image code
    __shared__ int32_t s_mark[kHeavyWaves][64];
    __shared__ int32_t s_total;
    __shared__ int32_t s_cnt[kHeavyWaves];        // listed chunks, then adjacent candidates, per wavefront
    __shared__ int32_t s_occ[kHeavyWaves];        // points of the adjacent candidates (COUNT)
    __shared__ int32_t s_chunk[kSegChunks];
    __shared__ uint64_t s_mask[MODE == kNbrFill ? kSegChunks : 1];
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    if (MODE == kNbrFill && totals[0] > cap) return;
    const int32_t nh = counters[1];
    const uint64_t below = (lane == 0) ? 0ull : (~0ull >> (64 - lane));
    for (int32_t h = blockIdx.x; h < nh; h += gridDim.x) {
        const int64_t A = heavy[h];
        const NbrLeaf f = nbr_leaf(t, A);
        if (w == 0) {
            const NbrRanges r0 = nbr_ranges<PER>(t, f, s_r);
            s_r[0][lane] = r0.lo;
            s_r[1][lane] = r0.pre;
            s_r[2][lane] = r0.code;
            if (lane == 0) s_total = r0.total;
        }
        __syncthreads();
        NbrRanges r;
        r.lo = s_r[0][lane];
        r.pre = s_r[1][lane];
        r.code = s_r[2][lane];
        r.total = __builtin_amdgcn_readfirstlane(s_total);
        const int32_t nch = (r.total + kChunk - 1) / kChunk;
        const int64_t out0 = MODE == kNbrFill ? nbr_start[A] : 0;
        int32_t written = 0, occ_sum = 0;
        for (int32_t seg = 0; seg < nch; seg += kSegChunks) {
            // ---- the chunks that may touch A, in order
            int32_t M = 0;
            const int32_t seg_end = min(nch, seg + kSegChunks);
            for (int32_t c = seg; c < seg_end; c += 64 * kHeavyWaves) {
                const int32_t ch = c + static_cast<int32_t>(threadIdx.x);
                const bool near = chunk_near<PER>(t, f, f.sA, r, ch) && ch < seg_end;
                const uint64_t bal = __ballot(near);
                if (lane == 0) s_cnt[w] = __popcll(bal);
                __syncthreads();
                int32_t at = M + __popcll(bal & below);
                for (int q = 0; q < kHeavyWaves; ++q) {
                    if (q < w) at += s_cnt[q];
                    M += s_cnt[q];
                }
                if (near) s_chunk[at] = ch;
                __syncthreads();
            }
            // ---- their adjacent candidates
            const int32_t per = (M + kHeavyWaves - 1) / kHeavyWaves;
            const int32_t j0 = min(M, w * per), j1 = min(M, j0 + per);
            int32_t cnt = 0;
            for (int32_t j = j0; j < j1; ++j) {
                const int32_t ch = __builtin_amdgcn_readfirstlane(s_chunk[j]);
                int32_t B = 0;
                int cB = 13;
                const bool adj = nbr_candidate<PER>(t, f, r, ch, s_mark[w], B, cB);
                const uint64_t bal = __ballot(adj);
                cnt += __popcll(bal);
                if (MODE == kNbrCount) {
                    if (adj) occ_sum += t.leaf_start[B + 1] - t.leaf_start[B];
                } else if (lane == 0) {
                    s_mask[j] = bal;
                }
            }
            if (lane == 0) s_cnt[w] = cnt;
            __syncthreads();
            int32_t pos = written;
            for (int q = 0; q < kHeavyWaves; ++q) {
                if (q < w) pos += s_cnt[q];
                written += s_cnt[q];
            }
            if (MODE == kNbrFill) {
                for (int32_t j = j0; j < j1; ++j) {
                    const int32_t ch = __builtin_amdgcn_readfirstlane(s_chunk[j]);
                    const uint64_t bal = s_mask[j];
                    const int32_t cidx = ch * kChunk + lane;
                    int32_t off;
                    int cB;
                    chunk_place<PER>(r, ch * kChunk, s_mark[w], off, cB);
                    if ((bal >> lane) & 1) {
                        const int64_t p = out0 + pos + __popcll(bal & below);
                        nbr_idx[p] = cidx + off;
                        if constexpr (PER) nbr_shift[p] = static_cast<int8_t>(cB);
                    }
                    pos += __popcll(bal);
                }
            }
            __syncthreads();   // s_cnt, s_chunk and s_mask are rewritten
        }
        if (MODE == kNbrCount) {
#pragma unroll
            for (int o = 32; o > 0; o >>= 1) occ_sum += __shfl_xor(occ_sum, o, 64);
            if (lane == 0) s_occ[w] = occ_sum;
            __syncthreads();
            if (threadIdx.x == 0) {
                int32_t all = 0;
                for (int q = 0; q < kHeavyWaves; ++q) all += s_occ[q];
                counts[A] = written;
                segs[A] = all;
            }
        }
        __syncthreads();   // the LDS ranges are rewritten for the next leaf
    }
}

// List starts: at most kStartGrid workgroups each sum the counts and segment
// lengths of `span` leaves, a multiple of kStartTile (k_nbr_sums), then scan
// their own span behind the sums before it (k_nbr_starts).  The starts are
// written only if all lists fit `cap` entries.
constexpr int kStartBlock = 256, kStartItems = 8, kStartTile = kStartBlock * kStartItems;
constexpr unsigned kStartGrid = 1024;

__device__ inline int64_t wave_sum(int64_t v) {
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
    return v;
}

__global__ __launch_bounds__(kStartBlock) void k_nbr_sums(const int32_t *__restrict__ counts,
                                                          const int32_t *__restrict__ segs, int64_t L, int64_t span,
                                                          int64_t *__restrict__ sums) {
    __shared__ int64_t s_w[2][kStartBlock / 64];
    const int64_t i0 = blockIdx.x * span, i1 = min(L, i0 + span);
    int64_t c = 0, g = 0;
    for (int64_t i = i0 + threadIdx.x; i < i1; i += kStartBlock) {
        c += counts[i];
        g += segs[i];
    }
    c = wave_sum(c);
    g = wave_sum(g);
    if ((threadIdx.x & 63) == 0) {
        s_w[0][threadIdx.x >> 6] = c;
        s_w[1][threadIdx.x >> 6] = g;
    }
    __syncthreads();
    if (threadIdx.x < 2) {
        int64_t v = 0;
        for (int q = 0; q < kStartBlock / 64; ++q) v += s_w[threadIdx.x][q];
        sums[threadIdx.x * kStartGrid + blockIdx.x] = v;
    }
}

__global__ __launch_bounds__(kStartBlock) void k_nbr_starts(const int32_t *__restrict__ counts, int64_t L,
                                                            int64_t span, const int64_t *__restrict__ sums,
                                                            int64_t cap, int64_t *__restrict__ nbr_start,
                                                            int64_t *__restrict__ totals) {
    constexpr int W = kStartBlock / 64;
    __shared__ int64_t s_w[3][W];
    const int t = threadIdx.x, lane = t & 63, w = t >> 6;
    int64_t before = 0, all = 0, seg = 0;
    for (unsigned q = t; q < gridDim.x; q += kStartBlock) {
        const int64_t v = sums[q];
        all += v;
        if (q < blockIdx.x) before += v;
        seg += sums[kStartGrid + q];
    }
    before = wave_sum(before);
    all = wave_sum(all);
    seg = wave_sum(seg);
    if (lane == 0) {
        s_w[0][w] = before;
        s_w[1][w] = all;
        s_w[2][w] = seg;
    }
    __syncthreads();
    before = all = seg = 0;
    for (int q = 0; q < W; ++q) {
        before += s_w[0][q];
        all += s_w[1][q];
        seg += s_w[2][q];
    }
    if (blockIdx.x == 0 && t == 0) {
        totals[0] = all;
        totals[1] = seg;
    }
    if (all > cap) return;
    if (blockIdx.x == 0 && t == 0) nbr_start[L] = all;
    const int64_t i1 = min(L, blockIdx.x * span + span);
    for (int64_t i0 = blockIdx.x * span; i0 < i1; i0 += kStartTile) {
        const int64_t base = i0 + t * kStartItems;
        int32_t v[kStartItems];
        int64_t s = 0;
#pragma unroll
        for (int k = 0; k < kStartItems; ++k) {
            v[k] = base + k < i1 ? counts[base + k] : 0;
            s += v[k];
        }
        int64_t inc = s;
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            const int64_t y = __shfl_up(inc, o, 64);
            if (lane >= o) inc += y;
        }
        __syncthreads();
        if (lane == 63) s_w[0][w] = inc;
        __syncthreads();
        int64_t p = before + inc - s;
        for (int q = 0; q < W; ++q) {
            if (q < w) p += s_w[0][q];
            before += s_w[0][q];
        }
#pragma unroll
        for (int k = 0; k < kStartItems; ++k) {
            if (base + k < i1) nbr_start[base + k] = p;
            p += v[k];
        }
    }
}

// The same for at most kOneStartMax leaves by one workgroup in one launch: it
// sums all counts first, then scans them.  16,384 leaves: 16 loads a thread,
// beside a launch of 5 us.
constexpr int64_t kOneStartMax = 16384;
__global__ __launch_bounds__(1024) void k_nbr_starts_one(const int32_t *__restrict__ counts,
                                                         const int32_t *__restrict__ segs, int64_t L, int64_t cap,
                                                         int64_t *__restrict__ nbr_start,
                                                         int64_t *__restrict__ totals) {
    __shared__ int64_t s_w[2][16];
    const int t = threadIdx.x, lane = t & 63, w = t >> 6;
    int64_t all = 0, seg = 0;
#pragma unroll 4
    for (int64_t i = t; i < L; i += 1024) {
        all += counts[i];
        seg += segs[i];
    }
    all = wave_sum(all);
    seg = wave_sum(seg);
    if (lane == 0) {
        s_w[0][w] = all;
        s_w[1][w] = seg;
    }
    __syncthreads();
    all = seg = 0;
    for (int q = 0; q < 16; ++q) {
        all += s_w[0][q];
        seg += s_w[1][q];
    }
    if (t == 0) {
        totals[0] = all;
        totals[1] = seg;
    }
    if (all > cap) return;
    if (t == 0) nbr_start[L] = all;
    int64_t before = 0;
    for (int64_t i0 = 0; i0 < L; i0 += 4096) {
        const int64_t base = i0 + 4 * t;
        int32_t v[4];
        int64_t s = 0;
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            v[k] = base + k < L ? counts[base + k] : 0;
            s += v[k];
        }
        int64_t inc = s;
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            const int64_t y = __shfl_up(inc, o, 64);
            if (lane >= o) inc += y;
        }
        __syncthreads();
        if (lane == 63) s_w[0][w] = inc;
        __syncthreads();
        int64_t p = before + inc - s;
        for (int q = 0; q < 16; ++q) {
            if (q < w) p += s_w[0][q];
            before += s_w[0][q];
        }
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            if (base + k < L) nbr_start[base + k] = p;
            p += v[k];
        }
    }
}

// Slots into the CSR lists: thread t = (A, s) moves entry s of a list that fit
// (and its image code, if slot_code is not null).  A heavy leaf's short list
// is not in its slots; k_neighbors_heavy writes it afterwards.
__device__ inline void compact_slot(int64_t t, const int32_t *__restrict__ counts, const int32_t *__restrict__ slots,
                                    const int8_t *__restrict__ slot_code, const int64_t *__restrict__ nbr_start,
                                    int64_t L, int32_t *__restrict__ nbr_idx, int8_t *__restrict__ nbr_shift) {
    const int64_t A = t / kNbrSlots;
    const int sidx = static_cast<int>(t % kNbrSlots);
    if (A >= L) return;
    const int32_t c = counts[A];
    if (c <= kNbrSlots && sidx < c) {
        nbr_idx[nbr_start[A] + sidx] = slots[t];
        if (slot_code) nbr_shift[nbr_start[A] + sidx] = slot_code[t];
    }
}

// After the starts: the first g_slots workgroups move the slots, the others
// search again for the lists over kNbrSlots entries.
template <bool PER>
__global__ __launch_bounds__(64 * kNbrWaves) void k_neighbors_finish(
    NbrTree t, const int32_t *__restrict__ counts, const int32_t *__restrict__ slots,
    const int8_t *__restrict__ slot_code, const int32_t *__restrict__ counters, const int32_t *__restrict__ heavy,
    const int64_t *__restrict__ totals, int64_t cap, const int64_t *__restrict__ nbr_start, uint32_t g_slots,
    int32_t *__restrict__ nbr_idx, int8_t *__restrict__ nbr_shift) {
    if (totals[0] > cap) return;
    if (blockIdx.x < g_slots)
        compact_slot(static_cast<int64_t>(blockIdx.x) * (64 * kNbrWaves) + threadIdx.x, counts, slots, slot_code,
                     nbr_start, t.Lt, nbr_idx, nbr_shift);
    else
        fill_long_lists<PER>(t, blockIdx.x - g_slots, gridDim.x - g_slots, counters, heavy, nbr_start, nbr_idx,
                             nbr_shift);
}

}  // namespace

int neighbor_dir_bits(int total_key_bits) { return total_key_bits < 18 ? total_key_bits : 18; }

p2p_status launch_key_directory(const uint64_t *leaf_key, int64_t L, int total_key_bits, int32_t *dir,
                                int32_t *counters, hipStream_t s) {
    const int db = neighbor_dir_bits(total_key_bits);
    const int64_t nb = (int64_t(1) << db) + 1;
    k_key_directory<<<grid_for(nb, 256), 256, 0, s>>>(leaf_key, L, db, total_key_bits - db, dir, counters);
    P2P_LAUNCH_CHECK();
    return P2P_OK;
}

namespace {
NbrTree make_tree(const uint64_t *leaf_key, const int8_t *leaf_level, const int32_t *leaf_start, int64_t L,
                  int key_bits, int inst_shift, const int32_t *dir, int total_key_bits, const NbrTargets *tg) {
    NbrTree t;
    t.leaf_key = leaf_key;
    t.leaf_level = leaf_level;
    t.leaf_start = leaf_start;
    t.dir = dir;
    t.L = L;
    t.tkey = tg ? tg->leaf_key : leaf_key;
    t.tlevel = tg ? tg->leaf_level : leaf_level;
    t.Lt = tg ? tg->L : L;
    t.key_bits = key_bits;
    t.inst_shift = inst_shift;
    t.dir_bits = neighbor_dir_bits(total_key_bits);
    t.dir_shift = total_key_bits - t.dir_bits;
    return t;
}
}  // namespace

size_t neighbor_sum_elems() { return 2 * kStartGrid; }

p2p_status launch_neighbors(const uint64_t *leaf_key, const int8_t *leaf_level, int64_t L, int key_bits,
                            int inst_shift, const int32_t *dir, int total_key_bits, const int32_t *leaf_start,
                            const NbrScratch &ws, int64_t cap, int64_t *nbr_start, int32_t *nbr_idx,
                            int8_t *nbr_shift, hipStream_t s, const NbrTargets *tg) {
    const NbrTree t = make_tree(leaf_key, leaf_level, leaf_start, L, key_bits, inst_shift, dir, total_key_bits, tg);
    const unsigned g_leaf = grid_for(t.Lt, kNbrWaves);
    // A list, and what is searched for it, holds no leaf twice in one image: few
    // source leaves leave no leaf heavy, and fewer no list over its slots
    const int64_t most = t.L * (ws.slot_code ? 27 : 1);
    const unsigned g_fill = most <= kNbrSlots ? 0 : g_leaf < kFillGrid ? g_leaf : kFillGrid;
    const unsigned g_heavy =
        most <= kHeavyCands ? 0 : t.Lt < kHeavyGrid ? static_cast<unsigned>(t.Lt) : kHeavyGrid;
#define P2P_NBR(PER)                                                                                              \
    k_neighbors_count<PER><<<g_leaf, 64 * kNbrWaves, 0, s>>>(t, ws.counts, ws.segs, ws.slots, ws.slot_code,      \
                                                             ws.counters, ws.heavy);                             \
    P2P_LAUNCH_CHECK();                                                                                           \
    if (g_heavy > 0)                                                                                              \
        k_neighbors_heavy<kNbrCount, PER><<<g_heavy, 64 * kHeavyWaves, 0, s>>>(                                   \
            t, ws.counts, ws.segs, ws.counters, ws.heavy, nullptr, 0, nullptr, nullptr, nullptr)
    if (t.Lt > 0) {
        if (ws.slot_code) { P2P_NBR(true); } else { P2P_NBR(false); }
        P2P_LAUNCH_CHECK();
    }
#undef P2P_NBR
    if (t.Lt <= kOneStartMax) {
        k_nbr_starts_one<<<1, 1024, 0, s>>>(ws.counts, ws.segs, t.Lt, cap, nbr_start, ws.totals);
    } else {
        const int64_t tiles = (t.Lt + kStartTile - 1) / kStartTile;
        const int64_t span = (tiles + kStartGrid - 1) / kStartGrid * kStartTile;
        const unsigned g = grid_for(t.Lt, static_cast<int>(span));
        k_nbr_sums<<<g, kStartBlock, 0, s>>>(ws.counts, ws.segs, t.Lt, span, ws.sums);
        P2P_LAUNCH_CHECK();
        k_nbr_starts<<<g, kStartBlock, 0, s>>>(ws.counts, t.Lt, span, ws.sums, cap, nbr_start, ws.totals);
    }
    P2P_LAUNCH_CHECK();
    if (t.Lt <= 0) return P2P_OK;
    const unsigned g_slots = grid_for(t.Lt * kNbrSlots, 64 * kNbrWaves);
#define P2P_NBR(PER)                                                                                            \
    k_neighbors_finish<PER><<<g_slots + g_fill, 64 * kNbrWaves, 0, s>>>(                                        \
        t, ws.counts, ws.slots, ws.slot_code, ws.counters, ws.heavy, ws.totals, cap, nbr_start, g_slots,        \
        nbr_idx, nbr_shift);                                                                                    \
    P2P_LAUNCH_CHECK();                                                                                         \
    if (g_heavy > 0)                                                                                            \
        k_neighbors_heavy<kNbrFill, PER><<<g_heavy, 64 * kHeavyWaves, 0, s>>>(                                  \
            t, nullptr, nullptr, ws.counters, ws.heavy, ws.totals, cap, nbr_start, nbr_idx, nbr_shift)
    if (ws.slot_code) { P2P_NBR(true); } else { P2P_NBR(false); }
#undef P2P_NBR
    P2P_LAUNCH_CHECK();
    return P2P_OK;
}

}  // namespace p2p
