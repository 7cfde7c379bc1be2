// Device prefix scan, key emission, stable LSD radix sort and tile ranges:
// the binning stage that turns per-pair tile rectangles into per-tile,
// front-to-back Gaussian lists (the tile partitioning of Sec. 4.1).
//
// Sort: reduce-then-scan LSD radix sort with 8-bit digits and a fixed grid (no
// inter-workgroup waits, so no forward-progress assumption). Each pass:
// per-block digit histograms -> per-digit exclusive scans over the blocks
// (digit offsets folded into the scatter prologue) -> scatter, where keys are ranked stably inside a 2048-key tile with wave64
// ballots (8 ballots give each lane the mask of lanes sharing its digit).
#include "kernels.h"
#include "swf_device.h"

namespace swf {

namespace {

constexpr int kThreads = 256;
constexpr int kWaves = kThreads / 64;
constexpr int kItems = 8;
constexpr int kTile = kThreads * kItems;  // keys per scatter tile
constexpr int kMaxGrid = 1024;

__device__ __forceinline__ unsigned lane_id() { return threadIdx.x & 63u; }

__device__ __forceinline__ uint64_t lanemask_lt() { return (1ull << lane_id()) - 1ull; }

// Inclusive scan across a wave64.
template <typename T>
__device__ __forceinline__ T wave_inclusive_scan(T v) {
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const T t = __shfl_up(v, o, 64);
        if ((int)lane_id() >= o) v += t;
    }
    return v;
}

// Exclusive scan across a block of W waves (256 threads by default); returns the block total in *tot.
template <typename T, int W = kWaves>
__device__ __forceinline__ T block_exclusive_scan(T v, T* lds /* W + 1 */, T* tot) {
    const T inc = wave_inclusive_scan(v);
    const int w = threadIdx.x >> 6;
    if (lane_id() == 63) lds[w] = inc;
    __syncthreads();
    if (threadIdx.x == 0) {
        T run = 0;
        for (int i = 0; i < W; ++i) {
            const T t = lds[i];
            lds[i] = run;
            run += t;
        }
        lds[W] = run;
    }
    __syncthreads();
    const T r = lds[w] + inc - v;
    *tot = lds[W];
    __syncthreads();
    return r;
}

// ---- exclusive scan of uint32 counts (3 kernels; 1 up to kScanSingleMax) ---
__global__ __launch_bounds__(kThreads) void scan_reduce_kernel(const uint32_t* __restrict__ in, int64_t n,
                                                               int64_t chunk, uint64_t* __restrict__ sums) {
    __shared__ uint64_t lds[kWaves + 1];
    const int64_t beg = (int64_t)blockIdx.x * chunk;
    const int64_t end = min(beg + chunk, n);
    uint64_t s = 0;
    for (int64_t i = beg + threadIdx.x; i < end; i += kThreads) s += in[i];
    uint64_t tot;
    block_exclusive_scan<uint64_t>(s, lds, &tot);
    if (threadIdx.x == 0) sums[blockIdx.x] = tot;
}

__global__ __launch_bounds__(kThreads) void scan_top_kernel(uint64_t* __restrict__ sums, int G,
                                                            uint64_t* __restrict__ total) {
    __shared__ uint64_t lds[kWaves + 1];
    uint64_t base = 0;
    for (int c = 0; c < G; c += kThreads) {
        const int i = c + threadIdx.x;
        const uint64_t v = i < G ? sums[i] : 0;
        uint64_t tot;
        const uint64_t ex = block_exclusive_scan<uint64_t>(v, lds, &tot);
        if (i < G) sums[i] = base + ex;
        base += tot;
    }
    if (threadIdx.x == 0) *total = base;
}

__global__ __launch_bounds__(kThreads) void scan_down_kernel(const uint32_t* __restrict__ in, int64_t n,
                                                             int64_t chunk, const uint64_t* __restrict__ sums,
                                                             uint32_t* __restrict__ out) {
    __shared__ uint64_t lds[kWaves + 1];
    const int64_t beg = (int64_t)blockIdx.x * chunk;
    const int64_t end = min(beg + chunk, n);
    uint64_t base = sums[blockIdx.x];
    // per-thread runs of kItems consecutive elements for coalescing-friendly reads
    for (int64_t t0 = beg; t0 < end; t0 += (int64_t)kThreads * kItems) {
        uint32_t v[kItems];
        uint64_t s = 0;
#pragma unroll
        for (int j = 0; j < kItems; ++j) {
            const int64_t i = t0 + (int64_t)threadIdx.x * kItems + j;
            v[j] = i < end ? in[i] : 0u;
            s += v[j];
        }
        uint64_t tot;
        uint64_t ex = block_exclusive_scan<uint64_t>(s, lds, &tot) + base;
#pragma unroll
        for (int j = 0; j < kItems; ++j) {
            const int64_t i = t0 + (int64_t)threadIdx.x * kItems + j;
            if (i < end) out[i] = (uint32_t)ex;
            ex += v[j];
        }
        base += tot;
    }
}

// Small inputs (n <= kScanSingleMax) in one launch: one 1024-thread workgroup
// stages the counts in LDS with coalesced loads, scans 16 consecutive counts
// per thread around one block scan, and writes the offsets back through LDS
// with coalesced stores (in and out may be the same array); writes the total.
constexpr int kScanSingleThreads = 1024;
constexpr int kScanSingleItems = 16;
constexpr int64_t kScanSingleMax = (int64_t)kScanSingleThreads * kScanSingleItems;  // 16384

__global__ __launch_bounds__(kScanSingleThreads) void scan_single_kernel(const uint32_t* in, int64_t n, uint32_t* out,
                                                                         uint64_t* __restrict__ total) {
    constexpr int W = kScanSingleThreads / 64;
    __shared__ uint4 s_v[kScanSingleMax / 4];
    __shared__ uint64_t lds[W + 1];
    uint32_t* sv = reinterpret_cast<uint32_t*>(s_v);
    const int t = (int)threadIdx.x;
#pragma unroll
    for (int k = 0; k < kScanSingleItems; ++k) {
        const int i = k * kScanSingleThreads + t;
        sv[i] = i < n ? in[i] : 0u;
    }
    __syncthreads();
    uint32_t v[kScanSingleItems];
#pragma unroll
    for (int q = 0; q < kScanSingleItems / 4; ++q) {
        const uint4 u = s_v[t * (kScanSingleItems / 4) + q];
        v[4 * q] = u.x;
        v[4 * q + 1] = u.y;
        v[4 * q + 2] = u.z;
        v[4 * q + 3] = u.w;
    }
    uint64_t s = 0;
#pragma unroll
    for (int j = 0; j < kScanSingleItems; ++j) s += v[j];
    uint64_t tot;
    uint64_t ex = block_exclusive_scan<uint64_t, W>(s, lds, &tot);  // ends with a barrier: every read above is done
#pragma unroll
    for (int q = 0; q < kScanSingleItems / 4; ++q) {
        uint4 u;
        u.x = (uint32_t)ex;
        ex += v[4 * q];
        u.y = (uint32_t)ex;
        ex += v[4 * q + 1];
        u.z = (uint32_t)ex;
        ex += v[4 * q + 2];
        u.w = (uint32_t)ex;
        ex += v[4 * q + 3];
        s_v[t * (kScanSingleItems / 4) + q] = u;
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < kScanSingleItems; ++k) {
        const int i = k * kScanSingleThreads + t;
        if (i < n) out[i] = sv[i];
    }
    if (t == 0) *total = tot;
}

// Culled pairs of a wave by reason (the reason a record with no tiles keeps in
// rect.y; 0 for pairs that are not culled): one atomic per reason and wave into
// cull[0] (non-finite or degenerate) and cull[1] (off the grid). Every lane of
// the wave must call it. cull may be null.
__device__ __forceinline__ void tally_culled(uint32_t why, unsigned long long* cull) {
    const uint64_t nf = __ballot(why == kCullNonFinite), og = __ballot(why == kCullOffGrid);
    if (cull && lane_id() == 0) {
        if (nf) atomicAdd(&cull[0], (unsigned long long)__popcll(nf));
        if (og) atomicAdd(&cull[1], (unsigned long long)__popcll(og));
    }
}

// ---- key emission -----------------------------------------------------------
// One thread per pair: one key per tile of the pair's rectangle, row-major.
// key = global tile (query * tiles + ty * TW + tx), or with full keys
// (global tile << 32 | depth bits); value = pair index.
template <bool kFull>
__global__ __launch_bounds__(kThreads) void emit_keys_kernel(const uint2* __restrict__ rect,
                                                             const uint32_t* __restrict__ count,
                                                             const uint32_t* __restrict__ offsets,
                                                             const uint32_t* __restrict__ dbits, int N, int64_t total,
                                                             int TW, int tiles, uint64_t capacity,
                                                             void* __restrict__ keys, uint32_t* __restrict__ vals,
                                                             uint32_t* __restrict__ status,
                                                             unsigned long long* __restrict__ cull) {
    const int64_t i = (int64_t)blockIdx.x * kThreads + threadIdx.x;
    const bool in = i < total;
    const uint32_t c = in ? count[i] : 0u;
    tally_culled(in && c == 0 ? rect[i].y : 0u, cull);
    if (!in || c == 0) return;
    const uint64_t off = offsets[i];
    if (off + c > capacity) {
        atomicOr(status, 1u);
        return;
    }
    const uint2 r = rect[i];
    const int tx0 = r.x & 0xffff, tx1 = r.x >> 16, ty0 = r.y & 0xffff, ty1 = r.y >> 16;
    // a wrapped rectangle (periodic azimuth, tx1 < tx0) spans columns tx0 .. TW-1, then 0 .. tx1
    const int ncol = tx1 >= tx0 ? tx1 - tx0 + 1 : TW - tx0 + tx1 + 1;
    const uint32_t q = (uint32_t)(i / N);
    const uint32_t base = q * (uint32_t)tiles;
    const uint32_t db = kFull ? dbits[i % N] : 0u;
    uint64_t o = off;
    for (int ty = ty0; ty <= ty1; ++ty) {
        for (int k = 0; k < ncol; ++k) {
            const int tx = tx0 + k < TW ? tx0 + k : tx0 + k - TW;
            const uint32_t gt = base + (uint32_t)(ty * TW + tx);
            if (kFull)
                reinterpret_cast<uint64_t*>(keys)[o] = ((uint64_t)gt << 32) | db;
            else
                reinterpret_cast<uint32_t*>(keys)[o] = gt;
            vals[o] = (uint32_t)i;
            ++o;
        }
    }
}

// ---- radix sort ---------------------------------------------------------------
// Key count and per-block chunk: from the host, or (n_dev != nullptr) read on
// the device as min(*n_dev, n) so that a captured graph needs no host sync.
__device__ __forceinline__ void sort_extent(const uint64_t* n_dev, int64_t& n, int64_t& chunk, int G) {
    if (n_dev) {
        const uint64_t d = *n_dev;
        n = (int64_t)(d < (uint64_t)n ? d : (uint64_t)n);
        chunk = (n + G - 1) / G;
        chunk = ((chunk + kTile - 1) / kTile) * kTile;
    }
}

template <typename K>
__global__ __launch_bounds__(kThreads) void radix_hist_kernel(const K* __restrict__ keys, int64_t n, int shift,
                                                              int64_t chunk, uint32_t* __restrict__ hist, int G,
                                                              const uint64_t* __restrict__ n_dev) {
    __shared__ uint32_t h[kWaves][256];
    sort_extent(n_dev, n, chunk, G);
    for (int i = threadIdx.x; i < kWaves * 256; i += kThreads) (&h[0][0])[i] = 0;
    __syncthreads();
    const int w = threadIdx.x >> 6;
    const int64_t beg = (int64_t)blockIdx.x * chunk;
    const int64_t end = min(beg + chunk, n);
    for (int64_t i = beg + threadIdx.x; i < end; i += kThreads) {
        const uint32_t d = (uint32_t)(keys[i] >> shift) & 255u;
        atomicAdd(&h[w][d], 1u);
    }
    __syncthreads();
    for (int d = threadIdx.x; d < 256; d += kThreads) {
        uint32_t s = 0;
#pragma unroll
        for (int k = 0; k < kWaves; ++k) s += h[k][d];
        hist[(size_t)d * G + blockIdx.x] = s;
    }
}

// Per-digit exclusive scan over the G block counts (digit-major histogram):
// block d scans hist[d][0..G) in place and writes the digit total.
__global__ __launch_bounds__(kThreads) void digit_scan_kernel(uint32_t* __restrict__ hist, int G,
                                                              uint32_t* __restrict__ dtot) {
    __shared__ uint32_t lds[kWaves + 1];
    uint32_t* h = hist + (size_t)blockIdx.x * G;
    uint32_t base = 0;
    for (int c = 0; c < G; c += kThreads) {
        const int i = c + threadIdx.x;
        const uint32_t v = i < G ? h[i] : 0u;
        uint32_t tot;
        const uint32_t ex = block_exclusive_scan<uint32_t>(v, lds, &tot);
        if (i < G) h[i] = base + ex;
        base += tot;
    }
    if (threadIdx.x == 0) dtot[blockIdx.x] = base;
}

template <typename K>
__global__ __launch_bounds__(kThreads) void radix_scatter_kernel(const K* __restrict__ kin,
                                                                 const uint32_t* __restrict__ vin,
                                                                 K* __restrict__ kout, uint32_t* __restrict__ vout,
                                                                 int64_t n, int shift, int64_t chunk,
                                                                 const uint32_t* __restrict__ hist, int G,
                                                                 const uint32_t* __restrict__ dtot,
                                                                 const uint64_t* __restrict__ n_dev) {
    sort_extent(n_dev, n, chunk, G);
    __shared__ uint32_t wcnt[kWaves][256];
    __shared__ uint32_t base[256];
    __shared__ uint32_t ttot[256];
    __shared__ uint32_t lds[kWaves + 1];
    const int w = threadIdx.x >> 6;
    {
        // digit offsets: exclusive scan of the digit totals
        static_assert(kThreads == 256, "one thread per digit");
        uint32_t tot;
        const uint32_t doff = block_exclusive_scan<uint32_t>(dtot[threadIdx.x], lds, &tot);
        base[threadIdx.x] = doff + hist[(size_t)threadIdx.x * G + blockIdx.x];
    }
    const int64_t beg = (int64_t)blockIdx.x * chunk;
    const int64_t end = min(beg + chunk, n);
    for (int64_t t0 = beg; t0 < end; t0 += kTile) {
        for (int i = threadIdx.x; i < kWaves * 256; i += kThreads) (&wcnt[0][0])[i] = 0;
        __syncthreads();
        K k[kItems];
        uint32_t v[kItems], dig[kItems], lr[kItems];
        bool ok[kItems];
#pragma unroll
        for (int j = 0; j < kItems; ++j) {
            const int64_t idx = t0 + (int64_t)(w * kItems + j) * 64 + lane_id();
            ok[j] = idx < end;
            k[j] = ok[j] ? kin[idx] : (K)0;
            v[j] = ok[j] ? vin[idx] : 0u;
            const uint32_t d = (uint32_t)(k[j] >> shift) & 255u;
            dig[j] = d;
            const uint64_t valid = __ballot(ok[j]);
            uint64_t match = valid;
#pragma unroll
            for (int b = 0; b < 8; ++b) {
                const bool bit = (d >> b) & 1u;
                const uint64_t bal = __ballot(bit && ok[j]);
                match &= bit ? bal : ~bal;
            }
            const uint32_t rank = (uint32_t)__popcll(match & lanemask_lt());
            const uint32_t cnt = (uint32_t)__popcll(match);
            uint32_t prev = 0;
            if (ok[j]) prev = wcnt[w][d];
            lr[j] = prev + rank;
            __builtin_amdgcn_wave_barrier();
            if (ok[j] && rank == 0) wcnt[w][d] = prev + cnt;
            __builtin_amdgcn_wave_barrier();
        }
        __syncthreads();
        for (int d = threadIdx.x; d < 256; d += kThreads) {
            uint32_t run = 0;
#pragma unroll
            for (int q = 0; q < kWaves; ++q) {
                const uint32_t c = wcnt[q][d];
                wcnt[q][d] = run;
                run += c;
            }
            ttot[d] = run;
        }
        __syncthreads();
#pragma unroll
        for (int j = 0; j < kItems; ++j) {
            if (ok[j]) {
                const uint32_t pos = base[dig[j]] + wcnt[w][dig[j]] + lr[j];
                kout[pos] = k[j];
                vout[pos] = v[j];
            }
        }
        __syncthreads();
        for (int d = threadIdx.x; d < 256; d += kThreads) base[d] += ttot[d];
        __syncthreads();
    }
}

// ---- binning: per-query stable counting sort by tile -----------------------
// Pairs are stored in (query, depth) order and a pair covers a tile at most
// once, so the list of a tile is the pairs covering it in pair order: the order
// of the full (tile, depth) sort, without keys in memory.
//   bin_hist:    block (j, q) counts, for every tile, the pairs
//                [j * pb, (j + 1) * pb) of query q that cover it, into its own
//                row: hist[(q * nbq + j) * stride + tile]
//   bin_offsets: per tile the exclusive prefix over the blocks, in place, the
//                tiles' first list positions and the entry count
//   bin_place:   block (j, q) writes its pairs into the tiles' lists; block
//                (0, q) also the tile ranges of query q
// A periodic azimuth has wrapped rectangles (tx1 < tx0: columns tx0 .. TW - 1,
// then 0 .. tx1).
struct BinGeom {
    int N, TW, TH, tiles;  // pairs per query and its tile grid (mixed batches: of the largest query; TW, TH unused)
    int stride;            // tiles per query, rounded up
    int chunk;             // (query, tile) columns whose first positions share a base
    bool whole;            // a block of bin_hist has all of its query's pairs, and writes its offsets as well
    int pb, nbq;           // pairs per block, blocks per query
    int cap;               // most pairs in a placement wave's row list and segment list
};

constexpr int kMaxTiles = 4096;   // tiles per query the binning path takes
constexpr int kHeldRows = 32;     // rows of a column that a thread of bin_offsets keeps in registers
constexpr int kPlaceWaves = 12;   // most waves of a placement block
constexpr int kSegCols = 8;       // tiles per column segment of the placement

// Blocks of 1024 pairs and lists of 640 up to 256 tiles (a row of a 90 x 360 grid meets ~430 of the 1024), of 2048
// and 512 beyond. Measured for the placement, us: 6.4M pairs at 90 x 360: 1024 / 640 109, 1024 / 512 118, 2048 158,
// 512 127; 32M pairs at 360 x 1440: 2048 / 512 1613, 4096 1899, 1024 2365, 2048 / 640 2629. What decides is how many
// waves the lists leave room for in LDS (24 per CU at the values taken), then how full the segment lists are.
// Halved (to 256 at least) while the batch has fewer than two blocks per compute unit: one query of 100k pairs is
// placed in 98 blocks at 1024 pairs, in 391 at 256.
//
// Columns: whole waves of tiles per query, but fours below 64 tiles, where most of a wave would be padding (1024
// queries of one tile: bin_offsets 7.0 us, 16.2 at 64 columns each). bin_offsets takes a column's rows (the blocks of
// its query) with one thread up to 8 rows, else with four, each of which keeps 32 rows in registers, or, past those
// 128 rows and while the columns are few, with 16, whose workgroups of 64 columns are spread over more compute units.
// us with 4 / 16: 100k pairs at 90 x 360, 1 query (391 rows) 25 / 10, 8 queries (98 rows) 11 / 11; 500k pairs at 360 x
// 1440, 1 query 29 / 15, 8 (16,896 columns) 20 / 17, 16 22 / 29, 64 121 / 202.
//
// A query of one block needs no column prefixes: bin_hist scans its own counts, the query is a chunk, and bin_offsets
// is not launched. Up to 128 queries, whose blocks count themselves off one by one at the end; us of bin_hist and
// bin_offsets / of bin_hist alone: 50 pairs of one tile, 1 query 7.8 / 5.2, 64 9.3 / 8.2, 256 10.0 / 13.7, 1024 11.4 /
// 39.9; 250 pairs of 138 tiles, 1 query 8.9 / 6.2, 64 12.5 / 8.6.
constexpr int kWholeQueries = 128;

BinGeom bin_geom(int64_t B, int N, int TW, int TH, int tiles) {
    BinGeom b;
    b.N = N;
    b.TW = TW;
    b.TH = TH;
    b.tiles = tiles;
    b.stride = tiles < 64 ? std::max(4, (tiles + 3) & ~3) : (tiles + 63) & ~63;
    b.pb = tiles <= 256 ? 1024 : 2048;
    while (b.pb > 256 && B * ((N + b.pb - 1) / b.pb) < 512) b.pb /= 2;
    b.nbq = std::max(1, (N + b.pb - 1) / b.pb);
    b.cap = std::min(b.pb, tiles <= 256 ? 640 : 512);
    b.whole = b.nbq == 1 && B <= kWholeQueries;
    b.chunk = b.whole ? b.stride : b.nbq > 4 * kHeldRows && B * b.stride <= 16384 ? 64 : 256;
    return b;
}

// The bins buffer. Column e = q * stride + tile; chunk e / G.chunk.
struct BinBufs {
    unsigned long long* ctot;  // list entries of a chunk of columns
    uint32_t* cbase;           // first list position of the chunk
    uint32_t* lstart;          // [B][stride] first list position of a column relative to its chunk
    uint32_t* hist;            // [B][nbq][stride]
};

int64_t bin_chunks(int64_t B, const BinGeom& G) { return (B * G.stride + G.chunk - 1) / G.chunk; }

size_t bin_words(int64_t B, const BinGeom& G) {
    const size_t ch = ((size_t)bin_chunks(B, G) + 1) & ~(size_t)1;
    return 3 * ch + (size_t)B * G.stride * (1 + (size_t)G.nbq);
}

BinBufs bin_bufs(uint32_t* bins, int64_t B, const BinGeom& G) {
    const size_t ch = ((size_t)bin_chunks(B, G) + 1) & ~(size_t)1;
    BinBufs b;
    b.ctot = reinterpret_cast<unsigned long long*>(bins);
    b.cbase = bins + 2 * ch;
    b.lstart = bins + 3 * ch;
    b.hist = b.lstart + (size_t)B * G.stride;
    return b;
}

// A query's pairs and tile grid for the binning kernels: uniform over a
// single-scene batch (G), from the batch's tables for a mixed one, whose
// geometry G (row stride, block size, blocks per query) covers its largest
// query: a smaller query leaves its extra blocks and tiles empty.
struct BinQuery {
    int N, TW, TH, tiles;
    size_t row0, tile0;  // first pair record, first global tile
};

template <bool kMix>
__device__ __forceinline__ BinQuery bin_query(const BinGeom& G, const MixBatch& mix, int q) {
    BinQuery b;
    if constexpr (kMix) {
        const MixQuery& a = mix.queries[q];
        const MixQuery& e = mix.queries[q + 1];
        b.N = e.pair_base - a.pair_base;  // 0 for the padding queries of a capacity-sized batch
        b.tiles = e.tile_base - a.tile_base;
        b.TW = mix.scenes[a.scene].TW;
        b.TH = b.tiles ? mix.scenes[a.scene].TH : 0;
        b.row0 = (size_t)a.pair_base;
        b.tile0 = (size_t)a.tile_base;
    } else {
        b.N = G.N;
        b.tiles = G.tiles;
        b.TW = G.TW;
        b.TH = G.TH;
        b.row0 = (size_t)q * G.N;
        b.tile0 = (size_t)q * G.tiles;
    }
    return b;
}

struct BinTotals {
    unsigned long long* total;  // entries of all lists
    uint64_t cap;               // 0: the host sizes the lists from the count
    unsigned long long* n_eff;
    uint32_t* status;
    uint32_t* done;             // zero at launch
    unsigned long long* host;   // pinned host copy of the total, or null
};

// Chunk `blk`'s total ct (thread 0's) is final. The last of the launch's nblk
// blocks to get here scans the chunk totals into the chunks' first positions and
// writes the counts. wsum: 16 words of LDS.
__device__ __forceinline__ void finish_totals(const BinBufs& bb, unsigned long long ct, int nblk, int blk,
                                              uint64_t* wsum, const BinTotals& T) {
    __shared__ int last;
    const int w = (int)threadIdx.x >> 6, W = (int)blockDim.x >> 6;
    if (threadIdx.x == 0) {
        __hip_atomic_store(&bb.ctot[blk], ct, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __threadfence();
        last = __hip_atomic_fetch_add(T.done, 1u, __ATOMIC_ACQ_REL, __HIP_MEMORY_SCOPE_AGENT) == (uint32_t)nblk - 1u;
    }
    __syncthreads();
    if (!last) return;
    __threadfence();
    uint64_t base = 0;
    for (int i0 = 0; i0 < nblk; i0 += (int)blockDim.x) {
        const int i = i0 + (int)threadIdx.x;
        const uint64_t x = i < nblk ? __hip_atomic_load(&bb.ctot[i], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : 0ull;
        const uint64_t ix = wave_inclusive_scan<uint64_t>(x);
        if (lane_id() == 63) wsum[w] = ix;
        __syncthreads();
        uint64_t before = 0, all = 0;
        for (int k = 0; k < W; ++k) {
            const uint64_t y = wsum[k];
            before += k < w ? y : 0ull;
            all += y;
        }
        if (i < nblk) bb.cbase[i] = (uint32_t)(base + before + ix - x);
        base += all;
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        *T.total = base;
        if (T.cap) {
            *T.n_eff = base <= T.cap ? base : 0ull;
            *T.status = base > T.cap ? 1u : 0u;
        }
        if (T.host) __hip_atomic_store(T.host, (unsigned long long)base, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
    }
}

// Tile counts of one block of pairs of one query. A rectangle adds one to every
// tile it covers, which is the two-dimensional running sum of +1 / -1 at its
// four corners: four LDS atomics per pair (eight for a wrapped rectangle)
// whatever its size, then one pass down the columns and a wave scan along each
// row. An atomic per covered tile instead (7 tiles per pair at 90 x 360, 20 at
// 180 x 720, every wave as long as its largest rectangle) took 44 us for 6.4M
// pairs at 90 x 360 and 140 us for 0.8M pairs at 180 x 720.
constexpr int kHistCells = kMaxTiles + 600;  // (TH + 1) (TW + 1) for TH TW <= kMaxTiles and TH, TW <= 512

// kWhole: the block has all of its query's pairs, so its counts are the query's.
// It scans them over the tiles (in the cells, 16 per thread at most) into the
// query's first positions, leaves zero column prefixes, and takes its part in
// the totals.
template <bool kMix, bool kWhole>
__global__ __launch_bounds__(kThreads) void bin_hist_kernel(const uint2* __restrict__ rect,
                                                            const uint32_t* __restrict__ count, BinGeom G,
                                                            BinBufs bb, unsigned long long* __restrict__ cull,
                                                            MixBatch mix, BinTotals T) {
    __shared__ int h[kHistCells];
    __shared__ uint64_t wsum[16];
    __shared__ uint32_t nculled[2];
    const int j = blockIdx.x, q = blockIdx.y;
    const BinQuery Q = bin_query<kMix>(G, mix, q);
    const int pitch = Q.TW + 1;
    for (int i = threadIdx.x; i < (Q.TH + 1) * pitch; i += kThreads) h[i] = 0;
    if (threadIdx.x < 2) nculled[threadIdx.x] = 0;
    __syncthreads();
    const int p_beg = j * G.pb, p_end = min(p_beg + G.pb, Q.N);
    uint32_t nf = 0, og = 0;  // culled pairs seen by this thread, by reason
    for (int p = p_beg + (int)threadIdx.x; p < p_end; p += kThreads) {
        const uint2 r = rect[Q.row0 + p];
        if (count[Q.row0 + p] == 0) {
            nf += r.y == kCullNonFinite;
            og += r.y == kCullOffGrid;
            continue;
        }
        const int tx0 = r.x & 0xffff, tx1 = r.x >> 16;
        int* top = h + (int)(r.y & 0xffff) * pitch;
        int* bot = h + ((int)(r.y >> 16) + 1) * pitch;
        atomicAdd(&top[tx0], 1);
        atomicAdd(&bot[tx0], -1);
        atomicAdd(&top[tx1 + 1], -1);
        atomicAdd(&bot[tx1 + 1], 1);
        if (tx1 < tx0) {  // wrapped: [0, tx1] and [tx0, TW)
            atomicAdd(&top[0], 1);
            atomicAdd(&bot[0], -1);
        }
    }
    if (nf) atomicAdd(&nculled[0], nf);
    if (og) atomicAdd(&nculled[1], og);
    __syncthreads();
    if (cull && threadIdx.x < 2 && nculled[threadIdx.x]) atomicAdd(&cull[threadIdx.x], (unsigned long long)nculled[threadIdx.x]);
    for (int c = threadIdx.x; c < Q.TW; c += kThreads) {
        int run = 0;
        for (int y = 0; y < Q.TH; ++y) {
            run += h[y * pitch + c];
            h[y * pitch + c] = run;
        }
    }
    __syncthreads();
    uint32_t* row = bb.hist + ((size_t)q * G.nbq + j) * G.stride;
    for (int y = threadIdx.x >> 6; y < Q.TH; y += kWaves) {
        int carry = 0;
        for (int c0 = 0; c0 < Q.TW; c0 += 64) {
            const int c = c0 + (int)lane_id();
            const int v = wave_inclusive_scan<int>(c < Q.TW ? h[y * pitch + c] : 0) + carry;
            if (c < Q.TW) {
                if constexpr (kWhole)
                    h[y * pitch + c] = v;
                else
                    row[y * Q.TW + c] = (uint32_t)v;
            }
            carry = __shfl(v, 63, 64);
        }
    }
    if constexpr (!kWhole) {
        for (int t = Q.tiles + (int)threadIdx.x; t < G.stride; t += kThreads) row[t] = 0u;
        return;
    }
    __syncthreads();
    // thread i takes the tiles from i per on, in row-major order
    const int per = (G.stride + kThreads - 1) / kThreads, t0 = (int)threadIdx.x * per;
    const int t1 = min(t0 + per, G.stride);
    auto cell = [&](int t) { return t < Q.tiles ? (uint32_t)h[t / Q.TW * pitch + t % Q.TW] : 0u; };
    uint32_t sum = 0;
    for (int t = t0; t < t1; ++t) sum += cell(t);
    const uint32_t inc = wave_inclusive_scan<uint32_t>(sum);
    const int w = (int)threadIdx.x >> 6;
    if (lane_id() == 63) wsum[w] = inc;
    __syncthreads();
    uint32_t run = inc - sum;
    unsigned long long all = 0;
    for (int k = 0; k < kWaves; ++k) {
        if (k < w) run += (uint32_t)wsum[k];
        all += wsum[k];
    }
    uint32_t* ls = bb.lstart + (size_t)q * G.stride;
    for (int t = t0; t < t1; ++t) {
        ls[t] = run;
        row[t] = 0u;
        run += cell(t);
    }
    __syncthreads();  // wsum is read
    finish_totals(bb, all, (int)gridDim.y, q, wsum, T);
}

// Block c: the kChunk columns from kChunk c on of the (query, tile) pairs. Per
// column the exclusive prefix over the query's nbq blocks, in place (the rows
// are cut into kGroups groups, summed, then rewritten; up to kHeldRows rows of a
// group stay in registers between), the columns' starts within the chunk and the
// chunk's total. The last block to finish (a counter the caller
// zeroed) scans the chunk totals into the chunks' first positions and writes
// the entry count, the count usable at a fixed capacity (total if it fits, else
// 0 with the overflow bit of the status word), and the count to the host. One
// launch; column prefixes, scan and count in five took 27 us per call at any
// size below 16k tiles.
template <int kChunk, int kGroups>
__global__ __launch_bounds__(kChunk* kGroups) void bin_offsets_kernel(BinBufs bb, BinGeom G, int64_t cols,
                                                                      BinTotals T) {
    __shared__ uint32_t part[kGroups][kChunk];
    __shared__ uint64_t wsum[16];
    constexpr int groups = kGroups;
    const int col = (int)threadIdx.x & (kChunk - 1), grp = (int)threadIdx.x / kChunk;
    const int w = (int)threadIdx.x >> 6;
    const int64_t e = (int64_t)blockIdx.x * kChunk + col;
    const bool in = e < cols;
    const int q = (int)((uint32_t)min(e, cols - 1) / (uint32_t)G.stride);
    const int R = (G.nbq + groups - 1) / groups;
    const int r0 = grp * R, r1 = in ? min(r0 + R, G.nbq) : r0;
    const size_t ld = (size_t)G.stride;
    uint32_t* h = bb.hist + (size_t)q * G.nbq * ld + (size_t)(e - (int64_t)q * G.stride);
    const bool held = R <= kHeldRows;
    uint32_t v[kHeldRows];
    uint32_t sum = 0;
    if (held) {
#pragma unroll
        for (int k = 0; k < kHeldRows; ++k) v[k] = r0 + k < r1 ? h[(size_t)(r0 + k) * ld] : 0u;
#pragma unroll
        for (int k = 0; k < kHeldRows; ++k) sum += v[k];
    } else {
        for (int r = r0; r < r1; r += kHeldRows) {
#pragma unroll
            for (int k = 0; k < kHeldRows; ++k) v[k] = r + k < r1 ? h[(size_t)(r + k) * ld] : 0u;
#pragma unroll
            for (int k = 0; k < kHeldRows; ++k) sum += v[k];
        }
    }
    part[grp][col] = sum;
    __syncthreads();
    uint32_t run = 0, tot = 0;
    for (int g = 0; g < groups; ++g) {
        if (g < grp) run += part[g][col];
        tot += part[g][col];
    }
    for (int r = r0; r < r1; r += kHeldRows) {
        if (!held)
#pragma unroll
            for (int k = 0; k < kHeldRows; ++k) v[k] = r + k < r1 ? h[(size_t)(r + k) * ld] : 0u;
#pragma unroll
        for (int k = 0; k < kHeldRows; ++k) {
            if (r + k < r1) h[(size_t)(r + k) * ld] = run;
            run += v[k];
        }
    }
    // the columns' starts within the chunk: the first kChunk threads hold one column each. Summed in 64 bits: 64
    // columns of 2^26 pairs are 2^32 entries, and only a total that shows it is refused (the positions are not used
    // then, so they may be cut to 32).
    uint64_t inc = 0;
    if (grp == 0) {
        inc = wave_inclusive_scan<uint64_t>(tot);
        if (lane_id() == 63) wsum[w] = inc;
    }
    __syncthreads();
    if (grp == 0) {
        uint64_t before = 0;
        for (int k = 0; k < w; ++k) before += wsum[k];
        if (in) bb.lstart[e] = (uint32_t)(before + inc - tot);
    }
    unsigned long long ct = 0;
    if (threadIdx.x == 0)
        for (int k = 0; k < kChunk / 64; ++k) ct += wsum[k];
    finish_totals(bb, ct, (int)gridDim.x, (int)blockIdx.x, wsum, T);
}

// base + the set bits of m below this lane
__device__ __forceinline__ uint32_t rank_below(uint64_t m, uint32_t base) {
    return __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, base));
}

// A pair of a placement block: first column (10 bits), last column (10 bits; a
// wrapped rectangle's runs past TW), index in the block (12 bits). kNoPair
// covers no column.
__device__ __forceinline__ uint32_t pack_pair(uint32_t c0, uint32_t c1, uint32_t id) {
    return c0 | (c1 << 10) | (id << 20);
}
constexpr uint32_t kNoPair = 1023u | (1022u << 10);

// Placement. The block's rectangles are staged in LDS; each wave takes tile
// rows of its own (row r, r + nw, ...), so no barrier and no atomic orders the
// writes. Per row it collects the pairs whose rectangle meets the row, in pair
// order (ballot compaction into its own LDS list); per segment of 8 columns the
// pairs of that list that meet the segment; then per 64 of those and per tile
// one ballot gives the covering lanes, which write their pair indices to
// consecutive list positions (the tile's next position is a scalar of the
// wave). Vector work per (64 candidates, tile): two instructions for the test,
// three for the rank and the store; a segment's candidates cover a given tile
// of it with probability ~1/4 on 1-12 px Gaussians, against ~1/20 without the
// two compactions. Finding each key's owner by binary search, ranking it by
// masks and storing it to a scattered 4-byte address (the earlier scheme; with
// several 512-tile segments, ranking by digit ballots) took 192 us for the 44M
// entries of 6.4M pairs at 90 x 360, 594 us for 15M entries at 180 x 720 and
// 2,923 us for 345M entries at 360 x 1440; this takes 102, 45 and 1,650 us,
// bound by instruction issue (at 360 x 1440 721M vector instructions, 71% of the
// cycles, and 688M scalar ones; 2.29 GB of HBM writes, 1.7 times the lists'
// bytes, at 1.4 TB/s).
template <bool kMix, bool kWrap>
__global__ __launch_bounds__(64 * kPlaceWaves) void bin_place_kernel(const uint2* __restrict__ rect,
                                                                     const uint32_t* __restrict__ count, BinGeom G,
                                                                     BinBufs bb,
                                                                     const unsigned long long* __restrict__ total,
                                                                     const unsigned long long* __restrict__ n_dev,
                                                                     uint32_t* __restrict__ vals,
                                                                     uint2* __restrict__ ranges, MixBatch mix) {
    extern __shared__ uint32_t s_dyn[];
    uint2* s_p = reinterpret_cast<uint2*>(s_dyn);  // (first row | rows << 16, packed pair); 0 rows: no tiles
    uint32_t* s_base = s_dyn + 2 * G.pb;           // next list position of every tile
    const int cap = G.cap;
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const int lane = (int)lane_id(), nw = (int)blockDim.x >> 6;
    uint32_t* s_row = s_base + G.stride + (size_t)wave * 2 * cap;  // the wave's lists of packed pairs
    uint32_t* s_seg = s_row + cap;
    const int j = blockIdx.x, q = blockIdx.y;
    const BinQuery Q = bin_query<kMix>(G, mix, q);
    const bool over = n_dev && *n_dev == 0;  // a fixed-capacity run that overflowed places nothing
    const int p_beg = j * G.pb, p_end = min(p_beg + G.pb, Q.N);
    const int np = max(p_end - p_beg, 0);
    const uint32_t e0 = (uint32_t)q * (uint32_t)G.stride;  // the query's first column
    if (j == 0) {
        const uint32_t all = gridDim.y * (uint32_t)G.stride;
        for (int t = threadIdx.x; t < Q.tiles; t += (int)blockDim.x) {
            const uint32_t e = e0 + (uint32_t)t, f = e + 1u;
            const uint32_t a = bb.lstart[e] + bb.cbase[e / (uint32_t)G.chunk];
            const uint32_t z = f < all ? bb.lstart[f] + bb.cbase[f / (uint32_t)G.chunk] : (uint32_t)*total;
            ranges[Q.tile0 + t] = !over && a < z ? make_uint2(a, z) : make_uint2(0u, 0u);
        }
    }
    if (over || np == 0) return;
    const uint32_t* hrow = bb.hist + ((size_t)q * G.nbq + j) * G.stride;
    for (int t = threadIdx.x; t < Q.tiles; t += (int)blockDim.x)
        s_base[t] = bb.lstart[e0 + t] + bb.cbase[(e0 + t) / (uint32_t)G.chunk] + hrow[t];
    const int nk = (np + 63) / 64;
    const int TW = Q.TW;
    for (int i = threadIdx.x; i < nk * 64; i += (int)blockDim.x) {
        uint2 p = make_uint2(0u, kNoPair);
        if (i < np && count[Q.row0 + p_beg + i]) {
            const uint2 r = rect[Q.row0 + p_beg + i];
            const uint32_t tx0 = r.x & 0xffff, tx1 = r.x >> 16, ty0 = r.y & 0xffff, ty1 = r.y >> 16;
            p = make_uint2(ty0 | ((ty1 - ty0 + 1u) << 16),
                           pack_pair(tx0, tx1 >= tx0 ? tx1 : tx1 + (uint32_t)TW, (uint32_t)i));
        }
        s_p[i] = p;
    }
    __syncthreads();
    const uint32_t v0 = (uint32_t)(Q.row0 + p_beg);
    constexpr int kU = 4;  // chunks read together
    for (int r = wave; r < Q.TH; r += nw) {
        for (int k = 0; k < nk;) {
            // the pairs of the next chunks that meet row r, at most a list's worth
            int n = 0;
            while (k < nk && n + 64 <= cap) {
                uint2 p[kU];
#pragma unroll
                for (int u = 0; u < kU; ++u) p[u] = s_p[min(k + u, nk - 1) * 64 + lane];
                int u0 = 0;  // chunks taken
#pragma unroll
                for (int u = 0; u < kU; ++u) {
                    if (k + u >= nk || n + 64 > cap) break;
                    const bool f = (uint32_t)r - (p[u].x & 0xffffu) < (p[u].x >> 16);
                    const uint64_t m = __ballot(f);
                    if (f) s_row[rank_below(m, (uint32_t)n)] = p[u].y;
                    n += __popcll(m);
                    u0 = u + 1;
                }
                k += u0;
            }
            // whole 64-pair chunks (n + 64 may pass the list: its last chunk is full then)
            if (n & 63) s_row[min(n + lane, n | 63)] = kNoPair;
            __builtin_amdgcn_wave_barrier();
            for (int c0 = 0; c0 < TW; c0 += kSegCols) {
                int ns = 0;
                for (int i = 0; i < n; i += 64 * kU) {
                    uint32_t p[kU];
#pragma unroll
                    for (int u = 0; u < kU; ++u) p[u] = i + 64 * u < n ? s_row[i + 64 * u + lane] : kNoPair;
#pragma unroll
                    for (int u = 0; u < kU; ++u) {
                        if (i + 64 * u >= n) break;
                        const uint32_t a = p[u] & 1023u, z = (p[u] >> 10) & 1023u;
                        bool f = a < (uint32_t)(c0 + kSegCols) && z >= (uint32_t)c0;
                        // the image one period to the left
                        if (kWrap) f = f || (z >= (uint32_t)(c0 + TW) && p[u] != kNoPair);
                        const uint64_t m = __ballot(f);
                        if (f) s_seg[rank_below(m, (uint32_t)ns)] = p[u];
                        ns += __popcll(m);
                    }
                }
                if (ns == 0) continue;
                if (ns & 63) s_seg[min(ns + lane, ns | 63)] = kNoPair;
                __builtin_amdgcn_wave_barrier();
                const int nc = min(kSegCols, TW - c0);
                uint32_t* sb = s_base + r * TW + c0;
                uint32_t vb = lane < nc ? sb[lane] : 0u;
                uint32_t b[kSegCols];
#pragma unroll
                for (int t = 0; t < kSegCols; ++t) b[t] = __builtin_amdgcn_readlane(vb, t);
                uint32_t next = s_seg[lane];
                for (int i = 0; i < ns; i += 64) {
                    const uint32_t p = next;
                    if (i + 64 < ns) next = s_seg[i + 64 + lane];
                    const uint32_t a = p & 1023u, w = ((p >> 10) & 1023u) + 1u - a;
                    const uint32_t d0 = (uint32_t)c0 - a;
                    const uint32_t v = v0 + (p >> 20);
#pragma unroll
                    for (int t = 0; t < kSegCols; ++t) {
                        bool f = d0 + (uint32_t)t < w;
                        if (kWrap) f = (f || d0 + (uint32_t)(t + TW) < w) && t < nc;
                        const uint64_t m = __ballot(f);
                        if (f) vals[rank_below(m, b[t])] = v;
                        b[t] += (uint32_t)__popcll(m);
                    }
                }
#pragma unroll
                for (int t = 0; t < kSegCols; ++t) vb = lane == t ? b[t] : vb;
                if (lane < nc) sb[lane] = vb;
                __builtin_amdgcn_wave_barrier();
            }
        }
    }
}

// ---- tile ranges -----------------------------------------------------------
__global__ void zero_ranges_kernel(uint2* __restrict__ r, int64_t m) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < m) r[i] = make_uint2(0u, 0u);
}

template <bool kFull>
__global__ void tile_ranges_kernel(const void* __restrict__ keys, int64_t n, uint2* __restrict__ r,
                                   const uint64_t* __restrict__ n_dev) {
    if (n_dev) {
        const uint64_t d = *n_dev;
        n = (int64_t)(d < (uint64_t)n ? d : (uint64_t)n);
    }
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    auto tile_of = [&](int64_t j) -> uint32_t {
        return kFull ? (uint32_t)(reinterpret_cast<const uint64_t*>(keys)[j] >> 32)
                     : reinterpret_cast<const uint32_t*>(keys)[j];
    };
    const uint32_t t = tile_of(i);
    if (i == 0 || tile_of(i - 1) != t) r[t].x = (uint32_t)i;
    if (i == n - 1 || tile_of(i + 1) != t) r[t].y = (uint32_t)(i + 1);
}

int radix_grid(int64_t n) {
    const int64_t tiles = (n + kTile - 1) / kTile;
    return (int)std::max<int64_t>(1, std::min<int64_t>(tiles, kMaxGrid));
}

template <typename K>
int radix_sort_t(K* keys, uint32_t* vals, K* kalt, uint32_t* valt, int64_t n, int begin_bit, int end_bit,
                 uint32_t* hist, hipStream_t st, const uint64_t* n_dev) {
    if (n <= 1 || end_bit <= begin_bit) return 0;
    const int G = radix_grid(n);
    uint32_t* dtot = hist + (size_t)256 * G;
    int64_t chunk = (n + G - 1) / G;
    chunk = ((chunk + kTile - 1) / kTile) * kTile;
    K* ki = keys;
    uint32_t* vi = vals;
    K* ko = kalt;
    uint32_t* vo = valt;
    int flips = 0;
    for (int shift = begin_bit; shift < end_bit; shift += 8) {
        radix_hist_kernel<K><<<G, kThreads, 0, st>>>(ki, n, shift, chunk, hist, G, n_dev);
        digit_scan_kernel<<<256, kThreads, 0, st>>>(hist, G, dtot);
        radix_scatter_kernel<K><<<G, kThreads, 0, st>>>(ki, vi, ko, vo, n, shift, chunk, hist, G, dtot, n_dev);
        std::swap(ki, ko);
        std::swap(vi, vo);
        flips ^= 1;
    }
    return flips;
}

}  // namespace

int scan_grid(int64_t n) {
    const int64_t per = (int64_t)kThreads * kItems;
    const int64_t g = (n + per - 1) / per;
    return (int)std::max<int64_t>(1, std::min<int64_t>(g, 4096));
}

size_t scan_scratch_bytes(int64_t n) { return sizeof(uint64_t) * (size_t)(scan_grid(n) + 1); }

void launch_exclusive_scan(const uint32_t* in, uint32_t* out, uint64_t* total, int64_t n, void* scratch,
                           hipStream_t st) {
    uint64_t* sums = reinterpret_cast<uint64_t*>(scratch);
    if (n <= 0) {
        launch_clear_u32(reinterpret_cast<uint32_t*>(total), 2, st);  // kernel, not a memset node
        return;
    }
    if (n <= kScanSingleMax) {  // e.g. the per-tile list totals of a batch: one launch instead of three
        scan_single_kernel<<<1, kScanSingleThreads, 0, st>>>(in, n, out, total);
        return;
    }
    const int G = scan_grid(n);
    int64_t chunk = (n + G - 1) / G;
    chunk = ((chunk + kThreads * kItems - 1) / (kThreads * kItems)) * (kThreads * kItems);
    scan_reduce_kernel<<<G, kThreads, 0, st>>>(in, n, chunk, sums);
    scan_top_kernel<<<1, kThreads, 0, st>>>(sums, G, total);
    scan_down_kernel<<<G, kThreads, 0, st>>>(in, n, chunk, sums, out);
}

void launch_emit_keys(const Records& r, const uint32_t* offsets, const uint32_t* dbits, int B, int N, const Grid& g,
                      uint64_t capacity, bool full_keys, void* keys, uint32_t* vals, uint32_t* status,
                      unsigned long long* cull, hipStream_t st) {
    const int64_t total = (int64_t)B * N;
    if (total <= 0) return;
    const unsigned blocks = (unsigned)((total + kThreads - 1) / kThreads);
    if (full_keys)
        emit_keys_kernel<true><<<blocks, kThreads, 0, st>>>(r.rect, r.count, offsets, dbits, N, total, g.TW, g.tiles,
                                                            capacity, keys, vals, status, cull);
    else
        emit_keys_kernel<false><<<blocks, kThreads, 0, st>>>(r.rect, r.count, offsets, dbits, N, total, g.TW,
                                                             g.tiles, capacity, keys, vals, status, cull);
}

size_t radix_scratch_bytes(int64_t n) { return sizeof(uint32_t) * 256 * ((size_t)radix_grid(n) + 1); }

int launch_radix_sort(void* keys, uint32_t* vals, void* kalt, uint32_t* valt, int64_t n, int key_bytes, int begin_bit,
                      int end_bit, void* scratch, hipStream_t st, const uint64_t* n_dev) {
    uint32_t* hist = reinterpret_cast<uint32_t*>(scratch);
    if (key_bytes == 8)
        return radix_sort_t<uint64_t>(reinterpret_cast<uint64_t*>(keys), vals, reinterpret_cast<uint64_t*>(kalt), valt,
                                      n, begin_bit, end_bit, hist, st, n_dev);
    return radix_sort_t<uint32_t>(reinterpret_cast<uint32_t*>(keys), vals, reinterpret_cast<uint32_t*>(kalt), valt, n,
                                  begin_bit, end_bit, hist, st, n_dev);
}

namespace {
__global__ void clear_u32_kernel(uint32_t* __restrict__ p, int n) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = 0u;
}
}  // namespace

namespace {
// Key count the sort may use after a fixed-capacity emission: the scan total
// if it fits, else 0 (the emission skipped pairs, so the key array has holes;
// the batch renders empty and the caller re-runs it with exact sizing).
// An overflow also sets bit 0 of the status word.
__global__ void effective_count_kernel(const uint64_t* __restrict__ total, uint64_t cap, uint64_t* __restrict__ n_eff,
                                       uint32_t* __restrict__ status) {
    if (threadIdx.x == 0 && blockIdx.x == 0) {
        const uint64_t t = *total;
        *n_eff = t <= cap ? t : 0ull;
        if (status) *status = t > cap ? 1u : 0u;  // stored, not or-ed: this sets the word for the launch's lists
    }
}
}  // namespace

void launch_effective_count(const uint64_t* total, uint64_t cap, uint64_t* n_eff, uint32_t* status, hipStream_t st) {
    effective_count_kernel<<<1, 64, 0, st>>>(total, cap, n_eff, status);
}

void launch_clear_u32(uint32_t* p, int n, hipStream_t st) {
    if (n > 0) clear_u32_kernel<<<(n + 255) / 256, 256, 0, st>>>(p, n);
}

void launch_tile_ranges(const void* keys, int key_bytes, int64_t n, int64_t n_gtiles, uint2* ranges, hipStream_t st,
                        const uint64_t* n_dev) {
    if (n_gtiles > 0) zero_ranges_kernel<<<(unsigned)((n_gtiles + 255) / 256), 256, 0, st>>>(ranges, n_gtiles);
    if (n <= 0) return;
    const unsigned blocks = (unsigned)((n + 255) / 256);
    if (key_bytes == 8)
        tile_ranges_kernel<true><<<blocks, 256, 0, st>>>(keys, n, ranges, n_dev);
    else
        tile_ranges_kernel<false><<<blocks, 256, 0, st>>>(keys, n, ranges, n_dev);
}

bool bin_fits(int B, int N, const Grid& g) { return B <= 65535 && g.tiles <= kMaxTiles; }

static BinGeom geom_of(int B, int N, const Grid& g) { return bin_geom(B, N, g.TW, g.TH, g.tiles); }
// Mixed batches: the geometry of the batch's largest query (max_n pairs, max_tiles tiles) for every query.
static BinGeom mix_geom(int B, int max_n, int max_tiles) { return bin_geom(B, max_n, 0, 0, max_tiles); }

size_t bin_entries(int B, int N, const Grid& g) { return bin_words(B, geom_of(B, N, g)); }
size_t mix_bin_entries(int B, int max_n, int max_tiles) { return bin_words(B, mix_geom(B, max_n, max_tiles)); }

// Tile counts, and the lists' first positions and totals
static void count_launch(const BinGeom& G, int B, const Records& r, uint32_t* bins, unsigned long long* cull,
                         const BinCount& c, hipStream_t st, const MixBatch* m) {
    BinTotals t;
    t.total = reinterpret_cast<unsigned long long*>(c.total);
    t.cap = c.cap;
    t.n_eff = reinterpret_cast<unsigned long long*>(c.n_eff);
    t.status = c.status;
    t.done = c.done;
    t.host = reinterpret_cast<unsigned long long*>(c.host);
    const BinBufs bb = bin_bufs(bins, B, G);
    const dim3 grid(G.nbq, B);
    if (m && G.whole)
        bin_hist_kernel<true, true><<<grid, kThreads, 0, st>>>(r.rect, r.count, G, bb, cull, *m, t);
    else if (m)
        bin_hist_kernel<true, false><<<grid, kThreads, 0, st>>>(r.rect, r.count, G, bb, cull, *m, t);
    else if (G.whole)
        bin_hist_kernel<false, true><<<grid, kThreads, 0, st>>>(r.rect, r.count, G, bb, cull, MixBatch{}, t);
    else
        bin_hist_kernel<false, false><<<grid, kThreads, 0, st>>>(r.rect, r.count, G, bb, cull, MixBatch{}, t);
    if (G.whole) return;
    const unsigned blocks = (unsigned)bin_chunks(B, G);
    const int64_t cols = (int64_t)B * G.stride;
    if (G.chunk == 64)
        bin_offsets_kernel<64, 16><<<blocks, 1024, 0, st>>>(bb, G, cols, t);
    else if (G.nbq > 8)
        bin_offsets_kernel<256, 4><<<blocks, 1024, 0, st>>>(bb, G, cols, t);
    else
        bin_offsets_kernel<256, 1><<<blocks, 256, 0, st>>>(bb, G, cols, t);
}

static void place_launch(const BinGeom& G, int B, int TH, bool wrap, const Records& r, uint32_t* bins,
                         const uint64_t* total, const uint64_t* n_dev, uint32_t* vals, uint2* ranges, hipStream_t st,
                         const MixBatch* m) {
    // waves: the tile rows dealt evenly over at most 12 (6 rows: 6 waves of one; 23 rows: 12 of two)
    const int rounds = (TH + kPlaceWaves - 1) / kPlaceWaves;
    const int nw = std::max(1, rounds ? (TH + rounds - 1) / rounds : 1);
    const size_t lds = 8 * (size_t)G.pb + 4 * (size_t)G.stride + (size_t)nw * 8 * G.cap;
    const dim3 grid(G.nbq, B);
    const auto* tot = reinterpret_cast<const unsigned long long*>(total);
    const auto* nd = reinterpret_cast<const unsigned long long*>(n_dev);
    const BinBufs bb = bin_bufs(bins, B, G);
    if (m)
        bin_place_kernel<true, false><<<grid, 64 * nw, lds, st>>>(r.rect, r.count, G, bb, tot, nd, vals, ranges, *m);
    else if (wrap)
        bin_place_kernel<false, true><<<grid, 64 * nw, lds, st>>>(r.rect, r.count, G, bb, tot, nd, vals, ranges,
                                                                  MixBatch{});
    else
        bin_place_kernel<false, false><<<grid, 64 * nw, lds, st>>>(r.rect, r.count, G, bb, tot, nd, vals, ranges,
                                                                   MixBatch{});
}

void launch_bin_count(const Records& r, int B, int N, const Grid& g, uint32_t* bins, unsigned long long* cull,
                      const BinCount& c, hipStream_t st) {
    count_launch(geom_of(B, N, g), B, r, bins, cull, c, st, nullptr);
}

void launch_bin_place(const Records& r, int B, int N, const Grid& g, uint32_t* bins, const uint64_t* total,
                      const uint64_t* n_dev, uint32_t* vals, uint2* ranges, hipStream_t st) {
    place_launch(geom_of(B, N, g), B, g.TH, g.wrap != 0, r, bins, total, n_dev, vals, ranges, st, nullptr);
}

bool mix_bin_fits(int B, int max_tiles) { return B <= 65535 && max_tiles <= kMaxTiles; }

void launch_mix_bin_count(const MixBatch& m, int max_n, int max_tiles, const Records& r, uint32_t* bins,
                          unsigned long long* cull, const BinCount& c, hipStream_t st) {
    if (m.B > 0) count_launch(mix_geom(m.B, max_n, max_tiles), m.B, r, bins, cull, c, st, &m);
}

void launch_mix_bin_place(const MixBatch& m, int max_n, int max_tiles, const Records& r, uint32_t* bins,
                          const uint64_t* total, const uint64_t* n_dev, uint32_t* vals, uint2* ranges,
                          hipStream_t st) {
    // the rows of the batch's grids are in its tables on the device: as many waves as a grid of max_tiles
    // squarish tiles has rows, the waves of a flatter grid idle
    if (m.B > 0)
        place_launch(mix_geom(m.B, max_n, max_tiles), m.B, max_tiles <= 256 ? 6 : 12, false, r, bins, total, n_dev,
                     vals, ranges, st, &m);
}

}  // namespace swf
