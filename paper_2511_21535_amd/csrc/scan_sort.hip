// Device-wide exclusive scan and stable LSD radix sort of (uint64 key, int32
// value) pairs.  Both are plain data-movement primitives used by tree
// binning, near-list construction and the restructure step.
#include <algorithm>

#include "p2p_internal.h"

namespace p2p {
namespace {

constexpr int kScanBlock = 256;
constexpr int kScanItems = 8;
constexpr int kScanTile = kScanBlock * kScanItems;   // 2048
constexpr int64_t kScanFusedBlocks = 4096;            // n up to 8M in two launches

// Exclusive scan of one value per thread across a 256-thread block.
// Returns the thread's exclusive prefix; *total receives the block sum.
template <class T>
__device__ T block_exclusive_scan(T v, T *lds /*[kScanBlock/64]*/, T *total) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    T x = v;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        T y = __shfl_up(x, o, 64);
        if (lane >= o) x += y;
    }
    if (lane == 63) lds[wave] = x;
    __syncthreads();
    T wave_off = 0, tot = 0;
#pragma unroll
    for (int w = 0; w < kScanBlock / 64; ++w) {
        T s = lds[w];
        if (w < wave) wave_off += s;
        tot += s;
    }
    __syncthreads();
    *total = tot;
    return wave_off + x - v;
}

template <class TI, class TO>
__global__ __launch_bounds__(kScanBlock) void k_scan_reduce(const TI *__restrict__ in, int64_t n,
                                                            TO *__restrict__ partial) {
    __shared__ TO lds[kScanBlock / 64];
    int64_t base = static_cast<int64_t>(blockIdx.x) * kScanTile + threadIdx.x * kScanItems;
    TO s = 0;
#pragma unroll
    for (int i = 0; i < kScanItems; ++i)
        if (base + i < n) s += static_cast<TO>(in[base + i]);
    TO tot;
    block_exclusive_scan<TO>(s, lds, &tot);
    if (threadIdx.x == 0) partial[blockIdx.x] = tot;
}

// Scans partial[0..nb) in place (exclusive) with a single block; partial[nb] = total.
template <class TO>
__global__ __launch_bounds__(kScanBlock) void k_scan_partials(TO *partial, int64_t nb) {
    __shared__ TO lds[kScanBlock / 64];
    TO carry = 0;
    for (int64_t c = 0; c < nb; c += kScanTile) {
        int64_t base = c + threadIdx.x * kScanItems;
        TO v[kScanItems];
        TO s = 0;
#pragma unroll
        for (int i = 0; i < kScanItems; ++i) {
            v[i] = (base + i < nb) ? partial[base + i] : TO(0);
            s += v[i];
        }
        TO tot;
        TO pre = block_exclusive_scan<TO>(s, lds, &tot) + carry;
#pragma unroll
        for (int i = 0; i < kScanItems; ++i) {
            if (base + i < nb) partial[base + i] = pre;
            pre += v[i];
        }
        carry += tot;
        __syncthreads();
    }
    if (threadIdx.x == 0) partial[nb] = carry;
}

// Down-sweep.  The block's offset is partial[blockIdx.x] when the partials
// were scanned by k_scan_partials (FUSED == false); with FUSED the block sums
// the raw block totals partial[0 .. blockIdx.x) itself (one launch fewer, for
// grids of up to kScanFusedBlocks blocks), and partial == nullptr means a
// single block with offset 0.
template <class TI, class TO, bool FUSED>
__global__ __launch_bounds__(kScanBlock) void k_scan_down(const TI *in, int64_t n,
                                                          const TO *__restrict__ partial,
                                                          int64_t nb, TO *out) {
    __shared__ TO lds[kScanBlock / 64];
    TO off = 0, tot;
    if (FUSED && partial) {
        for (int64_t i = threadIdx.x; i < blockIdx.x; i += kScanBlock) off += partial[i];
        block_exclusive_scan<TO>(off, lds, &tot);
        off = tot;
    } else if (!FUSED) {
        off = partial[blockIdx.x];
    }
    int64_t base = static_cast<int64_t>(blockIdx.x) * kScanTile + threadIdx.x * kScanItems;
    TO v[kScanItems];
    TO s = 0;
#pragma unroll
    for (int i = 0; i < kScanItems; ++i) {
        v[i] = (base + i < n) ? static_cast<TO>(in[base + i]) : TO(0);
        s += v[i];
    }
    TO pre = block_exclusive_scan<TO>(s, lds, &tot) + off;
    // every read of `in` by this block happened before the barrier inside the scan
#pragma unroll
    for (int i = 0; i < kScanItems; ++i) {
        if (base + i < n) out[base + i] = pre;
        pre += v[i];
    }
    if (threadIdx.x == 0) {
        if (FUSED && blockIdx.x == nb - 1) out[n] = off + tot;
        if (!FUSED && blockIdx.x == 0) out[n] = partial[nb];
    }
}

template <class TO>
__global__ void k_scan_empty(TO *out) { out[0] = 0; }

}  // namespace

size_t scan_ws_elems(int64_t n) { return static_cast<size_t>((n + kScanTile - 1) / kScanTile) + 2; }

template <class TI, class TO>
p2p_status exclusive_scan(const TI *in, TO *out, int64_t n, TO *scratch, hipStream_t s) {
    if (n <= 0) {
        k_scan_empty<TO><<<1, 1, 0, s>>>(out);
        P2P_LAUNCH_CHECK();
        return P2P_OK;
    }
    const int64_t nb = (n + kScanTile - 1) / kScanTile;
    const unsigned g = static_cast<unsigned>(nb);
    if (nb == 1) {
        k_scan_down<TI, TO, true><<<1, kScanBlock, 0, s>>>(in, n, nullptr, nb, out);
        P2P_LAUNCH_CHECK();
    } else if (nb <= kScanFusedBlocks) {
        k_scan_reduce<TI, TO><<<g, kScanBlock, 0, s>>>(in, n, scratch);
        P2P_LAUNCH_CHECK();
        k_scan_down<TI, TO, true><<<g, kScanBlock, 0, s>>>(in, n, scratch, nb, out);
        P2P_LAUNCH_CHECK();
    } else {
        k_scan_reduce<TI, TO><<<g, kScanBlock, 0, s>>>(in, n, scratch);
        P2P_LAUNCH_CHECK();
        k_scan_partials<TO><<<1, kScanBlock, 0, s>>>(scratch, nb);
        P2P_LAUNCH_CHECK();
        k_scan_down<TI, TO, false><<<g, kScanBlock, 0, s>>>(in, n, scratch, nb, out);
        P2P_LAUNCH_CHECK();
    }
    return P2P_OK;
}

template p2p_status exclusive_scan<int32_t, int64_t>(const int32_t *, int64_t *, int64_t, int64_t *,
                                                     hipStream_t);
template p2p_status exclusive_scan<int64_t, int64_t>(const int64_t *, int64_t *, int64_t, int64_t *,
                                                     hipStream_t);

// ------------------------------------------------------------------ sort --
// Stable LSD radix sort of (uint64 key, int32 value) pairs, 8 bits per pass.
// The passes are short, so what bounds them is the chain of launches and, in
// a tile, of the ranks: a tile is ranked by 16 wavefronts of one or four
// chunks of 64 keys each.  2^21 keys: scatter 15.6 us, counts 5.6, scan 4.7 a
// pass (four wavefronts of 16 chunks, and the generic scan of the counts,
// took 21.5, 7.8 and 9.4); 60-bit keys in four passes and sort_runs (15 us)
// instead of eight passes, 118 us instead of 310.
namespace {

constexpr int kSortThreads = 1024;
constexpr int kSortWaves = kSortThreads / 64;

// Lanes of the wavefront that hold the same digit, among the valid ones.
__device__ inline uint64_t digit_peers(uint32_t d, bool valid) {
    uint64_t peers = __ballot(valid);
#pragma unroll
    for (int b = 0; b < 8; ++b) {
        const uint64_t bal = __ballot((d >> b) & 1u);
        peers &= ((d >> b) & 1u) ? bal : ~bal;
    }
    return peers;
}
__device__ inline uint64_t lanes_below(int lane) { return lane == 0 ? 0ull : (~0ull >> (64 - lane)); }

// Exclusive prefix over the 256 digits, by the first four wavefronts (thread =
// digit); the other wavefronts pass through its barriers.
__device__ inline uint32_t digit_scan(uint32_t v, uint32_t *s_w) {
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    uint32_t inc = v;
    if (tid < 256) {
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            const uint32_t y = __shfl_up(inc, o, 64);
            if (lane >= o) inc += y;
        }
        if (lane == 63) s_w[wave] = inc;
    }
    __syncthreads();
    uint32_t woff = 0;
    if (tid < 256)
        for (int w = 0; w < wave; ++w) woff += s_w[w];
    __syncthreads();
    return woff + inc - v;
}

// Digit counts of a tile: hist[tile][digit] (SUM) or hist[digit][tile].
template <int K, bool SUM>
__global__ __launch_bounds__(kSortThreads) void k_radix_hist(const uint64_t *__restrict__ keys, int64_t n, int shift,
                                                             uint32_t *__restrict__ hist, int64_t ntiles) {
    __shared__ uint32_t h[4][256];
    const int tid = threadIdx.x;
    (&h[0][0])[tid] = 0;
    __syncthreads();
    const int64_t base = static_cast<int64_t>(blockIdx.x) * (kSortThreads * K);
#pragma unroll
    for (int c = 0; c < K; ++c) {
        const int64_t i = base + c * kSortThreads + tid;
        if (i < n) atomicAdd(&h[tid & 3][static_cast<uint32_t>(keys[i] >> shift) & 255u], 1u);
    }
    __syncthreads();
    if (tid < 256)
        hist[SUM ? static_cast<int64_t>(blockIdx.x) * 256 + tid : static_cast<int64_t>(tid) * ntiles + blockIdx.x] =
            h[0][tid] + h[1][tid] + h[2][tid] + h[3][tid];
}

// Exclusive scan of each digit's counts over the tiles, in place, and the
// digit's total: one workgroup per digit.
__global__ __launch_bounds__(kScanBlock) void k_radix_scan(uint32_t *__restrict__ hist, int64_t ntiles,
                                                           uint32_t *__restrict__ totals) {
    __shared__ uint32_t lds[kScanBlock / 64];
    uint32_t *__restrict__ h = hist + static_cast<int64_t>(blockIdx.x) * ntiles;
    uint32_t carry = 0;
    for (int64_t c = 0; c < ntiles; c += kScanTile) {
        const int64_t base = c + threadIdx.x * kScanItems;
        uint32_t v[kScanItems], s = 0;
#pragma unroll
        for (int i = 0; i < kScanItems; ++i) {
            v[i] = base + i < ntiles ? h[base + i] : 0u;
            s += v[i];
        }
        uint32_t tot;
        uint32_t pre = block_exclusive_scan<uint32_t>(s, lds, &tot) + carry;
#pragma unroll
        for (int i = 0; i < kScanItems; ++i) {
            if (base + i < ntiles) h[base + i] = pre;
            pre += v[i];
        }
        carry += tot;
    }
    if (threadIdx.x == 0) totals[blockIdx.x] = carry;
}

// The ranks of a tile's keys by one digit, called by kSortThreads threads: K
// chunks of 64 keys per wavefront in order.  Lanes holding the same digit are
// found with 8 ballots, the rank among them is a popcount, and a per-wave digit
// counter in LDS carries the running count from chunk to chunk; the counters
// are then scanned across the wavefronts and the digits.  pos[c] = the key's
// position in the tile sorted by the digit; dstart[d] = first position of digit
// d.
template <int K>
__device__ void tile_ranks(const uint64_t (&key)[K], const bool (&valid)[K], int shift, uint32_t (*cnt)[256],
                           uint32_t *dstart, uint32_t *s_w, uint32_t (&pos)[K]) {
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    for (int i = tid; i < kSortWaves * 256; i += kSortThreads) (&cnt[0][0])[i] = 0;
    __syncthreads();
    uint32_t dig[K];
#pragma unroll
    for (int c = 0; c < K; ++c) {
        const uint32_t d = static_cast<uint32_t>(key[c] >> shift) & 255u;
        const uint64_t peers = digit_peers(d, valid[c]);
        const uint32_t rank = static_cast<uint32_t>(__popcll(peers & lanes_below(lane)));
        const uint32_t base = valid[c] ? cnt[wave][d] : 0u;
        if (valid[c] && rank == 0) cnt[wave][d] = base + static_cast<uint32_t>(__popcll(peers));
        dig[c] = d;
        pos[c] = base + rank;
    }
    __syncthreads();
    uint32_t tot = 0;   // thread = digit: exclusive scan over the wavefronts
    if (tid < 256) {
#pragma unroll
        for (int w = 0; w < kSortWaves; ++w) {
            const uint32_t t = cnt[w][tid];
            cnt[w][tid] = tot;
            tot += t;
        }
    }
    const uint32_t first = digit_scan(tot, s_w);
    if (tid < 256) dstart[tid] = first;
    __syncthreads();
#pragma unroll
    for (int c = 0; c < K; ++c) pos[c] += dstart[dig[c]] + cnt[wave][dig[c]];
}

// The tile is rearranged in LDS by digit and written out in that order, so the
// keys of one digit leave as one contiguous, coalesced run.  With SUM every
// workgroup adds the counts of the tiles before it itself; otherwise they were
// scanned, and totals holds the digit totals.  FIRST: the values are the
// positions (vin is not read).
template <int K, bool SUM, bool FIRST>
__global__ __launch_bounds__(kSortThreads) void k_radix_scatter(
    const uint64_t *__restrict__ kin, const int32_t *__restrict__ vin, uint64_t *__restrict__ kout,
    int32_t *__restrict__ vout, int64_t n, int shift, const uint32_t *__restrict__ hist,
    const uint32_t *__restrict__ totals, int64_t ntiles) {
    constexpr int T = kSortThreads * K;
    __shared__ uint32_t cnt[kSortWaves][256];
    __shared__ uint32_t dstart[256], dbase[256], s_w[4];
    __shared__ uint64_t s_key[T];
    __shared__ int32_t s_val[T];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int64_t tbase = static_cast<int64_t>(blockIdx.x) * T;
    uint64_t key[K];
    int32_t val[K];
    bool valid[K];
    uint32_t pos[K];
#pragma unroll
    for (int c = 0; c < K; ++c) {
        const int64_t i = tbase + wave * (64 * K) + c * 64 + lane;
        valid[c] = i < n;
        key[c] = valid[c] ? kin[i] : 0ull;
        val[c] = FIRST ? static_cast<int32_t>(i) : (valid[c] ? vin[i] : 0);
    }
    // first output position of each digit of this tile: the digits before it, then the tiles before this one
    uint32_t tot = 0, off = 0;
    if (SUM) {
        uint32_t *sb = &cnt[0][0], *st = &cnt[4][0];   // four partial sums per digit
        uint32_t o = 0, a = 0;
        for (int64_t t = tid >> 8; t < ntiles; t += 4) {
            const uint32_t c = hist[t * 256 + (tid & 255)];
            a += c;
            if (t < blockIdx.x) o += c;
        }
        sb[tid] = o;
        st[tid] = a;
        __syncthreads();
        if (tid < 256) {
            off = sb[tid] + sb[tid + 256] + sb[tid + 512] + sb[tid + 768];
            tot = st[tid] + st[tid + 256] + st[tid + 512] + st[tid + 768];
        }
    } else if (tid < 256) {
        tot = totals[tid];
        off = hist[static_cast<int64_t>(tid) * ntiles + blockIdx.x];
    }
    off += digit_scan(tot, s_w);
    tile_ranks<K>(key, valid, shift, cnt, dstart, s_w, pos);
    if (tid < 256) dbase[tid] = off - dstart[tid];
#pragma unroll
    for (int c = 0; c < K; ++c)
        if (valid[c]) {
            s_key[pos[c]] = key[c];
            s_val[pos[c]] = val[c];
        }
    __syncthreads();
    const int tile_n = static_cast<int>(min<int64_t>(T, n - tbase));
    for (int i = tid; i < tile_n; i += kSortThreads) {
        const uint64_t k = s_key[i];
        const uint32_t p = dbase[static_cast<uint32_t>(k >> shift) & 255u] + static_cast<uint32_t>(i);
        kout[p] = k;
        vout[p] = s_val[i];
    }
}

// Few keys (the values are the positions): every key's place is the number of
// keys before it (smaller, or equal and earlier).  A workgroup holds all keys in LDS and places 16 of
// them, 64 threads counting for each; n <= kRankSortMax.  4096 keys: 9 us; one
// workgroup sorting them in LDS by four passes and their runs took 23 us, the
// 24 launches of eight radix passes 170 us.
constexpr int kRankKeys = 16;
constexpr int64_t kRankSortMax = 8192;
__global__ __launch_bounds__(kSortThreads) void k_rank_sort(const uint64_t *__restrict__ kin,
                                                            uint64_t *__restrict__ kout, int32_t *__restrict__ vout,
                                                            int n, TreeCounts *__restrict__ tc) {
    __shared__ uint64_t s_key[kRankSortMax];
    __shared__ int s_cnt[kSortWaves][kRankKeys];
    const int tid = threadIdx.x, q = tid & (kRankKeys - 1), seg = tid / kRankKeys;
    int bad = 0;
    for (int j = tid; j < n; j += kSortThreads) {
        const uint64_t k = kin[j];
        bad |= k == kBadKey ? 1 : 0;
        s_key[j] = k;
    }
    bad = __syncthreads_or(bad);
    if (blockIdx.x == 0 && tid == 0) *tc = TreeCounts{bad != 0 ? 1 : 0, 0, 0, 0, 0, 0};
    const int i = blockIdx.x * kRankKeys + q;
    const uint64_t key = i < n ? s_key[i] : 0ull;
    int cnt = 0;
    for (int j = seg; j < n; j += kSortThreads / kRankKeys) {
        const uint64_t k = s_key[j];
        cnt += k < key || (k == key && j < i) ? 1 : 0;
    }
    cnt += __shfl_xor(cnt, 16, 64);
    cnt += __shfl_xor(cnt, 32, 64);
    if ((tid & 63) < kRankKeys) s_cnt[tid >> 6][q] = cnt;
    __syncthreads();
    if (tid < kRankKeys && i < n) {
        int p = 0;
        for (int w = 0; w < kSortWaves; ++w) p += s_cnt[w][q];
        kout[p] = key;
        vout[p] = i;
    }
}

// A slot's run of equal bits from lo up, seen through a window of kRunMax keys on
// either side of the workgroup's kRunBlock slots (LDS, no key past either end).
__device__ inline void run_window(const uint64_t *__restrict__ k, int64_t n, uint64_t (&w)[kRunBlock + 2 * kRunMax]) {
    const int64_t b = static_cast<int64_t>(blockIdx.x) * kRunBlock;
    for (int i = threadIdx.x; i < kRunBlock + 2 * kRunMax; i += kRunBlock) {
        const int64_t j = b - kRunMax + i;
        w[i] = j >= 0 && j < n ? k[j] : ~0ull;   // no key has its top bit set
    }
    __syncthreads();
}
// Whether the run of window slot me holds more than kRunMax keys; else it is [a, e).
__device__ inline bool run_is_long(const uint64_t (&w)[kRunBlock + 2 * kRunMax], int me, int lo, int &a, int &e) {
    const uint64_t top = w[me] >> lo;
    a = me;
    e = me + 1;
    // the same kRunMax slots away: long, without counting it
    if ((w[me - kRunMax] >> lo) == top || (w[me + kRunMax] >> lo) == top) return true;
    while ((w[a - 1] >> lo) == top) --a;   // both end inside the window
    while ((w[e] >> lo) == top) ++e;
    return e - a > kRunMax;
}
// Long slots of the workgroup before this thread's (rank) and in all (total); the
// slots at which a long run begins, up to this one (begun) and in all (begins).
struct RunRank {
    int rank, total, begun, begins;
};
__device__ inline RunRank rank_long(bool is_long, bool begin) {
    __shared__ int s_c[2][kRunBlock / 64];
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    const uint64_t l = __ballot(is_long), f = __ballot(is_long && begin), below = lanes_below(lane);
    if (lane == 0) {
        s_c[0][wv] = __popcll(l);
        s_c[1][wv] = __popcll(f);
    }
    __syncthreads();
    RunRank r{static_cast<int>(__popcll(l & below)), 0, static_cast<int>(__popcll(f & (below | 1ull << lane))), 0};
    for (int q = 0; q < kRunBlock / 64; ++q) {
        if (q < wv) {
            r.rank += s_c[0][q];
            r.begun += s_c[1][q];
        }
        r.total += s_c[0][q];
        r.begins += s_c[1][q];
    }
    return r;
}

// Keys sorted by their bits from lo up: puts every run of equal upper bits in
// order of the whole key, ties in their present order: a slot counts its place
// in its run.  A run over kRunMax keys is left as it is and counted.
__global__ __launch_bounds__(kRunBlock) void k_sort_runs(const uint64_t *__restrict__ kin,
                                                         const int32_t *__restrict__ vin,
                                                         uint64_t *__restrict__ kout, int32_t *__restrict__ vout,
                                                         int64_t n, int lo, TreeCounts *__restrict__ tc, LongRuns lr) {
    __shared__ uint64_t w[kRunBlock + 2 * kRunMax];
    run_window(kin, n, w);
    const int64_t i = static_cast<int64_t>(blockIdx.x) * kRunBlock + threadIdx.x;
    const int me = threadIdx.x + kRunMax;
    const uint64_t key = w[me];
    bool is_long = false;
    if (i < n) {
        int a, e;
        is_long = run_is_long(w, me, lo, a, e);
        int64_t p = i;
        if (!is_long) {
            int r = a - me;
            for (int j = a; j < e; ++j) r += w[j] < key || (w[j] == key && j < me) ? 1 : 0;
            p = i + r;
        }
        kout[p] = key;
        vout[p] = vin[i];
    }
    const RunRank r = rank_long(is_long, (w[me - 1] >> lo) != (key >> lo));
    if (threadIdx.x == 0) {
        lr.slots[blockIdx.x] = r.total;
        lr.runs[blockIdx.x] = r.begins;
        if (r.total != 0) tc->long_found = 1;   // every writer writes the same
    }
}

// The keys of the runs that k_sort_runs left, in order: (number of the run, the
// bits below lo), their values and slots.  The runs are numbered by their slots, so
// the keys of a run stay within its slots when they are sorted.
__global__ __launch_bounds__(kRunBlock) void k_gather_runs(const uint64_t *__restrict__ kin,
                                                           const int32_t *__restrict__ vin, int64_t n, int lo,
                                                           LongRuns lr) {
    __shared__ uint64_t w[kRunBlock + 2 * kRunMax];
    if (lr.slots[blockIdx.x] == 0) return;   // the same for the whole workgroup
    run_window(kin, n, w);
    const int64_t i = static_cast<int64_t>(blockIdx.x) * kRunBlock + threadIdx.x;
    const int me = threadIdx.x + kRunMax;
    const uint64_t key = w[me];
    int a, e;
    const bool is_long = i < n && run_is_long(w, me, lo, a, e);
    const RunRank r = rank_long(is_long, (w[me - 1] >> lo) != (key >> lo));
    if (is_long) {
        const int64_t m = lr.slot_off[blockIdx.x] + r.rank;
        const uint64_t run = static_cast<uint64_t>(lr.run_off[blockIdx.x] + r.begun - 1);
        lr.keys[m] = run << lo | (key & ((1ull << lo) - 1ull));
        lr.vals[m] = vin[i];
        lr.slot[m] = static_cast<int32_t>(i);
    }
}

// Sorted, back to the slots, each of which holds its run's upper bits.
__global__ __launch_bounds__(kRunBlock) void k_scatter_runs(const uint64_t *__restrict__ ck,
                                                            const int32_t *__restrict__ cv,
                                                            const int32_t *__restrict__ slot, int32_t n_slots, int lo,
                                                            uint64_t *__restrict__ keys, int32_t *__restrict__ vals) {
    const int64_t m = static_cast<int64_t>(blockIdx.x) * kRunBlock + threadIdx.x;
    if (m >= n_slots) return;
    const int32_t i = slot[m];
    keys[i] = keys[i] >> lo << lo | (ck[m] & ((1ull << lo) - 1ull));
    vals[i] = cv[m];
}

// Three launches a pass (counts, scan, scatter), or two where the scatter's
// workgroups can add the counts of at most kSumTiles tiles themselves: 64 KB
// from L2 beside a launch of 4.7 us.
constexpr int64_t kSumTiles = 64;
constexpr int64_t kSmallTileMax = kSumTiles * kSortThreads;
int64_t sort_tiles(int64_t n) {
    const int64_t tile = n <= kSmallTileMax ? kSortThreads : 4 * kSortThreads;
    return (n + tile - 1) / tile;
}

template <int K, bool SUM>
p2p_status radix_pass(SortBufs &b, int64_t n, int shift, uint32_t *hist, hipStream_t s) {
    const int64_t ntiles = sort_tiles(n);
    const unsigned g = static_cast<unsigned>(ntiles);
    uint32_t *totals = hist + 256 * ntiles;
    k_radix_hist<K, SUM><<<g, kSortThreads, 0, s>>>(b.keys, n, shift, hist, ntiles);
    P2P_LAUNCH_CHECK();
    if (!SUM) {
        k_radix_scan<<<256, kScanBlock, 0, s>>>(hist, ntiles, totals);
        P2P_LAUNCH_CHECK();
    }
    if (b.vals)
        k_radix_scatter<K, SUM, false><<<g, kSortThreads, 0, s>>>(b.keys, b.vals, b.keys_tmp, b.vals_tmp, n, shift,
                                                                  hist, totals, ntiles);
    else
        k_radix_scatter<K, SUM, true><<<g, kSortThreads, 0, s>>>(b.keys, nullptr, b.keys_tmp, b.vals_tmp, n, shift,
                                                                 hist, totals, ntiles);
    P2P_LAUNCH_CHECK();
    return P2P_OK;
}

}  // namespace

size_t radix_hist_elems(int64_t n) {
    if (n <= 0) return 512;
    // tiles of 1024 keys up to kSmallTileMax, of 4096 beyond: the most of any size up to n
    const int64_t small = sort_tiles(n < kSmallTileMax ? n : kSmallTileMax);
    return static_cast<size_t>(256 * std::max(small, sort_tiles(n)) + 256);
}

p2p_status radix_sort_pairs(SortBufs &b, int64_t n, int lo, int hi, uint32_t *hist, hipStream_t s) {
    if (n <= 0) return P2P_OK;
    const bool sum = sort_tiles(n) <= kSumTiles;
    for (int shift = lo; shift < hi; shift += 8) {
        P2P_TRY(n <= kSmallTileMax ? (radix_pass<1, true>(b, n, shift, hist, s))
                : sum              ? (radix_pass<4, true>(b, n, shift, hist, s))
                                   : (radix_pass<4, false>(b, n, shift, hist, s)));
        b.swap();
    }
    return P2P_OK;
}

bool rank_sort_fits(int64_t n) { return n <= kRankSortMax; }

p2p_status rank_sort_pairs(SortBufs &b, int64_t n, TreeCounts *tc, hipStream_t s) {
    if (n <= 0) return P2P_OK;
    if (!rank_sort_fits(n) || b.vals) return fail(P2P_EINVAL, "rank sort: too many keys, or values of their own");
    k_rank_sort<<<grid_for(n, kRankKeys), kSortThreads, 0, s>>>(b.keys, b.keys_tmp, b.vals_tmp, static_cast<int>(n),
                                                               tc);
    P2P_LAUNCH_CHECK();
    b.swap();
    return P2P_OK;
}

p2p_status sort_runs(SortBufs &b, int64_t n, int lo, TreeCounts *tc, const LongRuns &lr, hipStream_t s) {
    if (n <= 0) return P2P_OK;
    k_sort_runs<<<grid_for(n, kRunBlock), kRunBlock, 0, s>>>(b.keys, b.vals, b.keys_tmp, b.vals_tmp, n, lo, tc, lr);
    P2P_LAUNCH_CHECK();
    b.swap();
    return P2P_OK;
}

p2p_status sort_long_runs(SortBufs &b, int64_t n, int lo, const LongRuns &lr, int32_t n_runs, int32_t n_slots,
                          uint32_t *hist, hipStream_t s) {
    if (n_runs <= 0) return P2P_OK;
    P2P_TRY((exclusive_scan<int32_t, int64_t>(lr.slots, lr.slot_off, run_blocks(n), lr.scan, s)));
    P2P_TRY((exclusive_scan<int32_t, int64_t>(lr.runs, lr.run_off, run_blocks(n), lr.scan, s)));
    k_gather_runs<<<grid_for(n, kRunBlock), kRunBlock, 0, s>>>(b.keys, b.vals, n, lo, lr);
    P2P_LAUNCH_CHECK();
    SortBufs c{lr.keys, b.keys_tmp, lr.vals, b.vals_tmp, nullptr};
    int hi = lo;
    while ((int64_t(1) << (hi - lo)) < n_runs) ++hi;
    P2P_TRY(radix_sort_pairs(c, n_slots, 0, hi, hist, s));
    k_scatter_runs<<<grid_for(n_slots, kRunBlock), kRunBlock, 0, s>>>(c.keys, c.vals, lr.slot, n_slots, lo, b.keys,
                                                                      b.vals);
    P2P_LAUNCH_CHECK();
    return P2P_OK;
}

}  // namespace p2p
