// Device helpers of the column path of the Helmholtz product (helmholtz_cols.hip,
// helmholtz_split.hip): the columns of an instance are its (target box,
// right-hand side) pairs, numbered box * nrhs + rhs and cut into tiles.
#pragma once

#include "p2p_internal.h"

namespace p2p {
namespace {

// G(dd) = e^{i kh sqrt(dd)} / (4 pi sqrt(dd)) at unit spacing, dd the squared
// distance of two points of near boxes in spacings (0..147); zero for dd = 0,
// which leaves the point itself out.
constexpr int kDistances = 148;
__device__ inline double2 green(double kh, int dd) {
    if (dd == 0) return make_double2(0.0, 0.0);
    const double r = sqrt(static_cast<double>(dd)), a = 1.0 / (4.0 * 3.14159265358979323846 * r);
    double sn, cs;
    sincos(kh * r, &sn, &cs);
    return make_double2(cs * a, sn * a);
}
// k h of table tab, from the kernel arguments or the uploaded array.
__device__ inline double table_kh(const HelmInline &inl, const double *__restrict__ kh_dev, int tab) {
    if (inl.n_grids == 0) return kh_dev[tab];
    double kh = 0.0;
    // compile-time indices only, so the argument array stays in the kernel arguments
#pragma unroll
    for (int i = 0; i < kInlineGrids; ++i)
        if (i == tab) kh = inl.kh[i];
    return kh;
}
// dd between target i of a box and source s of the box at offset o =
// (ox+1) + 3 (oy+1) + 9 (oz+1); points in local Morton order.
__device__ inline int near_distance(int o, int s, int i) {
    const int od[3] = {o % 3 - 1, (o / 3) % 3 - 1, o / 9 - 1};
    int dd = 0;
#pragma unroll
    for (int d = 0; d < 3; ++d) {
        const int li = ((i >> d) & 1) | (((i >> (d + 3)) & 1) << 1);
        const int ls = ((s >> d) & 1) | (((s >> (d + 3)) & 1) << 1);
        const int diff = li - (ls + 4 * od[d]);
        dd += diff * diff;
    }
    return dd;
}

// Rows of nrhs entries into sorted order, sorted[s] = q[perm[s]], by workgroup b
// of 256 threads: four entries a thread, in flight together.  I holds the entry
// indices; entries past the end repeat the last (same bytes, same place).
constexpr int kPermuteEntries = 4 * 256;
template <class T, class I>
__device__ inline void permute_entries(const T *__restrict__ q, const int32_t *__restrict__ perm, I entries, I nrhs,
                                       T *__restrict__ sorted, I b) {
    const I base = b * kPermuteEntries + threadIdx.x;
    T v[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        const I e = min(base + 256 * k, entries - 1), row = e / nrhs;
        v[k] = q[static_cast<uint64_t>(perm[row]) * nrhs + (e - row * nrhs)];
    }
#pragma unroll
    for (int k = 0; k < 4; ++k) sorted[min(base + 256 * k, entries - 1)] = v[k];
}

// The column tile of workgroup b: the instance's first leaf, the tile's first
// column c0 among the instance's columns (column = box * nrhs + right-hand
// side) and column count cnt, the G table and 1/h of the instance (sc in
// float; sc64 in double from inl.iscale64 or inst_h, when inst_h or the inline
// parameters are given).  Called by whole wavefronts: with uploaded parameters
// the lanes compare b with the instances' first tiles, so the search is one
// round of loads for up to 64 instances.
struct ColTile {
    int32_t leaf0, cnt, tab;
    int64_t c0;
    float sc;
    double sc64;
};
template <int CB>
__device__ inline ColTile col_tile(const HelmInline &inl, const HelmTiles &ht, int32_t nrhs,
                                   const int32_t *__restrict__ inst_table, const float *__restrict__ inst_scale,
                                   const double *__restrict__ inst_h, int32_t b) {
    ColTile t;
    t.sc = 1.f;
    t.sc64 = 1.0;
    t.tab = 0;
    int32_t tf = 0, lf = 0, lf1 = 0;
    if (inl.n_grids > 0) {
#pragma unroll
        for (int i = 0; i < kInlineGrids; ++i)
            if (i < inl.n_grids && b >= inl.tile_first[i]) {
                tf = inl.tile_first[i];
                lf = inl.leaf_first[i];
                lf1 = inl.leaf_first[i + 1];
                t.tab = inl.itab[i];
                t.sc = inl.iscale[i];
                t.sc64 = inl.iscale64[i];
            }
    } else {
        int g = -1;   // instances whose first tile is at most b, less one
        for (int32_t i0 = 0; i0 < ht.n_grids; i0 += 64) {
            const int32_t i = i0 + static_cast<int32_t>(threadIdx.x & 63);
            g += __popcll(__ballot(i < ht.n_grids && ht.tile_first[min(i, ht.n_grids - 1)] <= b));
        }
        tf = ht.tile_first[g];
        lf = ht.leaf_first[g];
        lf1 = ht.leaf_first[g + 1];
        t.tab = inst_table[g];
        if (inst_scale) t.sc = inst_scale[g];
        if (inst_h) t.sc64 = 1.0 / inst_h[g];
    }
    t.leaf0 = lf;
    t.c0 = static_cast<int64_t>(CB) * (b - tf);
    t.cnt = static_cast<int32_t>(min<int64_t>(CB, static_cast<int64_t>(lf1 - lf) * nrhs - t.c0));
    return t;
}

// The (offset, box) map of a tile in LDS: the first source row of every
// (offset, box) from the near lists of the tile's boxes (one contiguous run of
// the CSR; -1 where the box has no such neighbour), and each box's first
// sorted target row.
struct ColMapView {
    int64_t *row;         // [27][cap]
    int64_t *nstart;      // [cap + 1]: list start of each box
    uint64_t *key;        // [cap]: local Morton key
    int64_t *rstart;      // [cap]: segment start (redundant layout, box grain)
    int32_t *tstart;      // [cap]: first sorted target row
    int32_t *present;     // [27]: 1 where some box of the tile has a neighbour at the offset
    int32_t cap;
};
template <int CB>
struct ColMap {
    int64_t row[27 * CB], nstart[CB + 1], rstart[CB];
    uint64_t key[CB];
    int32_t tstart[CB], present[27];
    __device__ ColMapView view() { return {row, nstart, key, rstart, tstart, present, CB}; }
};
// The same in dynamic LDS, from `base`.
__host__ __device__ inline size_t col_map_bytes(int cap) {
    return (static_cast<size_t>(27 + 3) * cap + 1) * 8 + static_cast<size_t>(cap + 27) * 4;
}
__device__ inline ColMapView col_map_view(void *base, int cap) {
    ColMapView m;
    m.cap = cap;
    m.row = static_cast<int64_t *>(base);
    m.nstart = m.row + 27 * cap;
    m.rstart = m.nstart + cap + 1;
    m.key = reinterpret_cast<uint64_t *>(m.rstart + cap);
    m.tstart = reinterpret_cast<int32_t *>(m.key + cap);
    m.present = m.tstart + cap;
    return m;
}

// Fills m for the cnt boxes from leaf A0; called by the whole workgroup (T threads), ends with a
// barrier.  Each column's list start, key, segment start and first target row
// come in one round of loads; then the entries, two per thread with their
// loads issued together: at most 27 per box, so a round of 2 T covers the tiles of
// up to 32 boxes; one of 128 (many columns, one right-hand side) takes four.
template <bool RED, int T>
__device__ void col_map(const ColMapView &m, int key_bits, int32_t A0, int32_t cnt, const int32_t *__restrict__ leaf_start,
                        const uint64_t *__restrict__ leaf_key, const int64_t *__restrict__ nbr_start,
                        const int32_t *__restrict__ nbr_idx, const int64_t *__restrict__ red_start,
                        const int64_t *__restrict__ red_row) {
    const int tid = threadIdx.x;
    const uint64_t local_mask = (1ull << (3 * key_bits)) - 1ull;
    for (int i = tid; i < 27 * m.cap; i += T) m.row[i] = -1;
    if (tid < 27) m.present[tid] = 0;
    for (int k = tid; k <= cnt; k += T) {
        // all four loads in flight at once (entry cnt only needs the list end)
        const int32_t a = A0 + min(k, cnt - 1);
        const int64_t ns = nbr_start[A0 + k];
        const uint64_t key = leaf_key[a];
        const int64_t rs = (RED && !red_row) ? red_start[a] : 0;
        const int32_t ts = leaf_start[a];
        m.nstart[k] = ns;
        if (k < cnt) {
            m.key[k] = key & local_mask;
            m.rstart[k] = rs;
            m.tstart[k] = ts;
        }
    }
    __syncthreads();
    const int64_t e_lo = m.nstart[0], e_hi = m.nstart[cnt];
    for (int64_t e0 = e_lo + tid; e0 < e_hi; e0 += 2 * T) {
        int64_t ev[2] = {e0, e0 + T};
        int32_t Bv[2];
        uint64_t lB[2];
        int64_t rv[2];
#pragma unroll
        for (int p = 0; p < 2; ++p) Bv[p] = nbr_idx[ev[p] < e_hi ? ev[p] : e0];
#pragma unroll
        for (int p = 0; p < 2; ++p) {
            lB[p] = leaf_key[Bv[p]] & local_mask;
            rv[p] = RED ? (red_row ? red_row[ev[p] < e_hi ? ev[p] : e0] : 0) : static_cast<int64_t>(leaf_start[Bv[p]]);
        }
#pragma unroll
        for (int p = 0; p < 2; ++p) {
            const int64_t e = ev[p];
            if (e >= e_hi) break;
            int j = 0, jh = cnt - 1;   // the box whose list holds e
            while (j < jh) {
                const int mid = (j + jh + 1) >> 1;
                if (m.nstart[mid] <= e) j = mid; else jh = mid - 1;
            }
            const uint64_t lA = m.key[j];
            const int ox = (static_cast<int>(p2pd::compact3(lB[p])) - static_cast<int>(p2pd::compact3(lA))) / 4;
            const int oy =
                (static_cast<int>(p2pd::compact3(lB[p] >> 1)) - static_cast<int>(p2pd::compact3(lA >> 1))) / 4;
            const int oz =
                (static_cast<int>(p2pd::compact3(lB[p] >> 2)) - static_cast<int>(p2pd::compact3(lA >> 2))) / 4;
            const int o = (ox + 1) + 3 * (oy + 1) + 9 * (oz + 1);
            m.present[o] = 1;   // every writer stores the same value
            m.row[o * m.cap + j] = (RED && !red_row) ? m.rstart[j] + 64 * (e - m.nstart[j]) : rv[p];
        }
    }
    __syncthreads();
}

// Column li of a tile: its box (an index into the map) and right-hand side,
// the first leaf A0 of the tile's boxes and their number.
struct ColLane {
    int32_t A0, boxes, box, rhs;
};
template <bool ONE>
__host__ __device__ inline ColLane col_lane(const ColTile &t, int32_t nrhs, int li) {
    ColLane l;
    if constexpr (ONE) {
        l.A0 = t.leaf0 + static_cast<int32_t>(t.c0);
        l.boxes = t.cnt;
        l.box = li;
        l.rhs = 0;
    } else {
        const int64_t b0 = t.c0 / nrhs;
        const int32_t r0 = static_cast<int32_t>(t.c0 - b0 * nrhs);   // < nrhs; r0 + 15 may pass 2^31
        l.A0 = t.leaf0 + static_cast<int32_t>(b0);
        l.boxes = static_cast<int32_t>((static_cast<int64_t>(r0) + t.cnt - 1) / nrhs) + 1;
        const uint32_t c = static_cast<uint32_t>(r0) + static_cast<uint32_t>(li < t.cnt ? li : t.cnt - 1);
        l.box = static_cast<int32_t>(c / static_cast<uint32_t>(nrhs));
        l.rhs = static_cast<int32_t>(c - static_cast<uint32_t>(l.box) * static_cast<uint32_t>(nrhs));
    }
    return l;
}

// The right-hand side of a wavefront's first column where nrhs is a multiple of
// 16 and its 16 columns are those of one box, from any lane's rhs.  A wavefront
// past the tile's last column holds that column in every lane; from the start of
// its group of 16 its loads stay inside the box's rows all the same.
__host__ __device__ inline int32_t uni_first_rhs(int32_t rhs) { return rhs & ~15; }

}  // namespace
}  // namespace p2p
