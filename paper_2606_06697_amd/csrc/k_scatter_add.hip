// Guarded scatter-add dst[idx[i], :] += src[i, :] (kernel memory guard of AgileOS Section V-E),
// organised so that heavily repeated destination rows (the hot rows of a Zipf-distributed
// embedding gradient) neither serialize on atomics nor pay one atomic row-update per index.
//
// Sorted path (large calls). Rows that pass the guard's fast test (index readable, source row
// wholly inside its allowed prefix, destination row inside the binding's row interval) get a
// 32-bit key, their destination row's offset inside that interval; every other row gets the
// largest key. A stable LSD radix sort (8-bit digits; per pass: per-tile digit histograms, their
// exclusive scan, a stable scatter that ranks a tile's keys with wave ballots and regroups them
// by digit in LDS, so that each digit's keys leave the tile as one contiguous run; a pass whose
// digit is the same for every key is skipped on the device) orders (key, position) pairs by
// destination row, position ascending. Groups of lanes (a wave for wide rows) then walk tiles of
// sorted entries and sum the source rows of each run of equal keys in position order. A run that
// lies inside one workgroup's tiles owns its destination row and adds with a plain
// read-modify-write, a run that crosses workgroups adds with one atomic per element. When the caller
// promises a destination of +0.0 rows (scatter-add into zeros), an owned run stores (+0.0 + its sum)
// without reading the row. Rows that failed the fast test follow in a separate kernel that checks
// every element exactly (denied loads read zero, denied stores are dropped) and counts denials as
// the other data-dependent guarded kernels do.
//
// Chunk path (smaller calls, or destination intervals too large for 32-bit keys): one kernel, whose
// workgroups sort 64 to 1,024 consecutive indices each in LDS and add each row of the chunk once, with
// one atomic per element; rows outside the interval are checked per element. The order of the atomics
// is not fixed: a row with indices in three or more chunks may differ in its last bits from call to call.
//
// Measured against an earlier chunk path of 2,048 indices a workgroup (one CU in use for every 2,048
// rows) and a reduce with a wave per row of any width (Zipf indices, 4,096-2^20 destination rows):
//   rows x columns       before     now
//     5,000 x 64         312 us     13 us   (chunks)
//    50,000 x 32          85 us     26 us   (chunks)
//   131,072 x 64         131 us     41 us   (chunks)
//   1,048,576 x 32       190 us    125 us   (sorted)
//   1,048,576 x 256      358 us    327 us   (sorted; the reduce alone 297 -> 265)
#include <type_traits>

#include "launch.h"

namespace agile {

constexpr int SAU = 8;               // source rows in flight per lane group
// Rows per chunk: the least power of two from 64 to 1024 that makes at most 32 chunks. Small chunks
// spread over more CUs, but add a hot row's sum in more steps, each of them rounded: relative
// error of the sum for 16,384 x 32 Zipf indices 5.4e-8 with 32 chunks, 6.5e-8 with 64 (6.1e-8 for
// chunks of 2,048 added in pieces of 32). Time 21 us against 23 us with 64 chunks of 256.
constexpr uint64_t SA_CHUNKS = 32;
constexpr uint64_t SA_SLOW = ~0ull;  // key of rows that fail the guard's fast test

template <int W>
struct FloatOf;
template <>
struct FloatOf<4> {
    using F = float;
    using E = uint32_t;
};
template <>
struct FloatOf<8> {
    using F = double;
    using E = uint64_t;
};

// Columns c0, c0 + step, ... of a row that failed the fast test: every element checked exactly, atomics
// for the allowed ones.
template <bool GUARD, int W>
__device__ inline void add_row_exact(uint8_t* dst, uint64_t rb, const int64_t* idx,
                                     const uint8_t* src, uint64_t r, const RowsGuard& rg,
                                     uint32_t c0, uint32_t step, FaultAcc& acc) {
    using F = typename FloatOf<W>::F;
    const uint64_t D = rb / W;
    const bool iok = !GUARD || r < rg.ki;
    if (!iok && c0 == 0) acc.note((r * D) << 2);
    const int64_t iv = iok ? idx[r] : 0;
    uint8_t* drow = dst + (uint64_t)iv * rb;
    for (uint64_t col = c0; col < D; col += step) {
        const uint64_t es = r * D + col;
        const bool sok = !GUARD || es < rg.kc;
        if (!sok) acc.note((es << 2) | 1u);
        // the source element is read only where its sum may be stored
        if (!GUARD || elem_ok(rg.g, iv, rb, col, W))
            unsafeAtomicAdd(reinterpret_cast<F*>(drow + col * W),
                            sok ? reinterpret_cast<const F*>(src)[es] : (F)0.0);
        else
            acc.note((es << 2) | 2u);
    }
}

// Adds a run's sum to its destination row: columns col, col + G, ... of the row with key `key`.
template <bool GUARD, int W, int EPL>
__device__ __forceinline__ void add_sum(uint8_t* dst, uint64_t rb, int64_t rlo, uint64_t key,
                                        uint64_t col, uint32_t G, uint64_t D,
                                        const typename FloatOf<W>::F (&sum)[EPL]) {
    using F = typename FloatOf<W>::F;
    const int64_t r = GUARD ? (int64_t)(key + (uint64_t)rlo) : (int64_t)(key ^ 0x8000000000000000ull);
    F* d = reinterpret_cast<F*>(dst + (uint64_t)r * rb) + col;
#pragma unroll
    for (int q = 0; q < EPL; ++q)
        if (col + q * G < D) unsafeAtomicAdd(d + q * G, sum[q]);
}

// CH consecutive indices per workgroup, sorted by destination row in LDS: each wave sorts 64 of them
// (a key counts the keys before it), then each key finds its place among the other sorted blocks by
// binary search (CH = 1024 takes two barriers and about 160 LDS reads a thread). Groups of 2^glog2 lanes walk segments of
// `seg` sorted entries side by side: SAU source rows are loaded at once and summed in position order
// while the destination stays the same. A run that spans segments is put together in LDS by the
// group in whose segment it ends, so that each row of the chunk gets one atomic add per element: a
// row's atomics are served one after another (about 25 ns for 64 bytes), and a hot row of a Zipf
// batch has a run in every chunk. A lane holds EPL columns a group's width apart, so that each
// atomic instruction covers whole lines.
template <bool GUARD, int W, int EPL, int CH, int TB>
__global__ __launch_bounds__(TB) void k_scatter_add(DevLog* log, uint8_t* dst, uint64_t rb,
                                                    const int64_t* idx, const uint8_t* src,
                                                    uint64_t n, RowsGuard rg, int logon,
                                                    uint32_t glog2, FinishOf<GUARD> fin) {
    using F = typename FloatOf<W>::F;
    constexpr uint32_t NB = CH / 64;
    __shared__ __align__(16) uint64_t kin[CH], kblk[CH];  // keys as they came, and each 64 sorted
    __shared__ uint64_t skey[CH];
    __shared__ uint16_t spos[CH];
    __shared__ F part[EPL][TB];  // sum of each segment's last run, if the next one goes on with it
    const uint64_t D = rb / W;
    const RowGuard g = rg.g;
    const uint32_t tid = threadIdx.x;
    const uint32_t G = 1u << glog2, lir = tid & (G - 1), grp = tid >> glog2;
    const uint32_t ng = TB >> glog2;
    const uint32_t seg = CH / ng > (uint32_t)SAU ? CH / ng : (uint32_t)SAU;  // ng * seg >= CH
    FaultAcc acc;
    for (uint64_t c0 = (uint64_t)blockIdx.x * CH; c0 < n; c0 += (uint64_t)gridDim.x * CH) {
        const uint32_t cnt = (uint32_t)(n - c0 < CH ? n - c0 : CH);
        // destination keys: offset of the row inside the binding's row interval, or SA_SLOW
        uint64_t key = SA_SLOW;
        if (tid < CH) {
            const uint64_t i = c0 + tid;
            if (tid < cnt) {
                if (GUARD) {
                    const int64_t iv = i < rg.nfast ? idx[i] : 0;
                    if (i < rg.nfast && g.rlo <= iv && iv <= g.rhi) key = (uint64_t)iv - (uint64_t)g.rlo;
                } else {
                    key = (uint64_t)idx[i] ^ 0x8000000000000000ull;  // order-preserving
                }
            }
            kin[tid] = key;
        }
        __syncthreads();
        const uint32_t blk = tid >> 6, lane = tid & 63u;
        uint32_t rank = 0;
        if (tid < CH) {
#pragma unroll 4
            for (uint32_t j = 0; j < 64; j += 2) {
                const ulonglong2 k2 = *reinterpret_cast<const ulonglong2*>(&kin[blk * 64 + j]);
                rank += (k2.x < key || (k2.x == key && j < lane)) ? 1u : 0u;
                rank += (k2.y < key || (k2.y == key && j + 1 < lane)) ? 1u : 0u;
            }
            if (NB > 1) kblk[blk * 64 + rank] = key;
        }
        if (NB > 1) {
            __syncthreads();
            if (tid < CH) {
#pragma unroll 4
                for (uint32_t o = 0; o < NB; ++o) {
                    if (o == blk) continue;
                    // keys of block o that come before: less, or equal in an earlier block
                    uint32_t p = 0;
#pragma unroll
                    for (uint32_t step = 32; step; step >>= 1) {
                        const uint64_t k = kblk[o * 64 + p + step - 1];
                        p += (k < key || (k == key && o < blk)) ? step : 0u;
                    }
                    const uint64_t k = kblk[o * 64 + p];
                    rank += p + ((k < key || (k == key && o < blk)) ? 1u : 0u);
                }
            }
        }
        if (tid < CH) {
            skey[rank] = key;
            spos[rank] = (uint16_t)tid;
        }
        __syncthreads();
        const uint32_t e0 = grp * seg;
        uint32_t e1 = e0 + seg < cnt ? e0 + seg : cnt;
        if (GUARD && e0 < cnt && skey[e1 - 1] == SA_SLOW) {
            // the segment ends where the rows that failed the fast test begin
            uint32_t lo = e0;
            for (uint32_t hi = e1 - 1; lo < hi;) {
                const uint32_t mid = (lo + hi) / 2;
                if (skey[mid] == SA_SLOW) hi = mid;
                else lo = mid + 1;
            }
            e1 = lo;
        }
        const bool some = e0 < e1;
        const uint64_t k0 = some ? skey[e0] : SA_SLOW, klast = some ? skey[e1 - 1] : SA_SLOW;
        const bool from_prev = some && e0 > 0 && skey[e0 - 1] == k0;
        const bool to_next = some && e1 < cnt && skey[e1] == klast;
        for (uint64_t cb = 0; cb < D; cb += (uint64_t)G * EPL) {
            F sum[EPL], head[EPL];  // head: the end of a run that earlier segments began
            bool ends_here = false, first = true;
            uint64_t cur = k0;
#pragma unroll
            for (int q = 0; q < EPL; ++q) sum[q] = (F)-0.0;
            for (uint32_t b = e0; b < e1; b += SAU) {
                F v[SAU][EPL];
#pragma unroll
                for (int u = 0; u < SAU; ++u) {
                    const uint32_t e = b + u;
                    if (e < e1) {
                        const F* sp = reinterpret_cast<const F*>(src + (c0 + spos[e]) * rb) + cb + lir;
#pragma unroll
                        for (int q = 0; q < EPL; ++q)
                            if (cb + lir + q * G < D) v[u][q] = sp[q * G];
                    }
                }
#pragma unroll
                for (int u = 0; u < SAU; ++u) {
                    const uint32_t e = b + u;
                    if (e >= e1) break;
                    const uint64_t k = skey[e];
                    if (k != cur) {
                        if (first && from_prev) {
                            ends_here = true;
#pragma unroll
                            for (int q = 0; q < EPL; ++q) head[q] = sum[q];
                        } else {
                            add_sum<GUARD, W, EPL>(dst, rb, g.rlo, cur, cb + lir, G, D, sum);
                        }
                        first = false;
                        cur = k;
#pragma unroll
                        for (int q = 0; q < EPL; ++q) sum[q] = (F)-0.0;
                    }
#pragma unroll
                    for (int q = 0; q < EPL; ++q) sum[q] += v[u][q];
                }
            }
            if (some) {
                if (to_next) {
#pragma unroll
                    for (int q = 0; q < EPL; ++q) part[q][tid] = sum[q];
                } else if (first && from_prev) {
                    ends_here = true;
#pragma unroll
                    for (int q = 0; q < EPL; ++q) head[q] = sum[q];
                } else {
                    add_sum<GUARD, W, EPL>(dst, rb, g.rlo, cur, cb + lir, G, D, sum);
                }
            }
            __syncthreads();
            if (ends_here) {
                uint32_t p = grp - 1;  // the segment in which the run begins
                while (p > 0 && skey[p * seg] == k0 && skey[p * seg - 1] == k0) --p;
                F run[EPL];
#pragma unroll
                for (int q = 0; q < EPL; ++q) run[q] = (F)-0.0;
                for (; p < grp; ++p)
#pragma unroll
                    for (int q = 0; q < EPL; ++q) run[q] += part[q][(p << glog2) + lir];
#pragma unroll
                for (int q = 0; q < EPL; ++q) run[q] += head[q];
                add_sum<GUARD, W, EPL>(dst, rb, g.rlo, k0, cb + lir, G, D, run);
            }
            __syncthreads();
        }
        // Rows that failed the fast test sort last, before the unused slots of a last chunk. A group of lanes
        // per row (33,000 rows of 1 / 16 / 64 floats, all denied, 18 / 24 / 44 us; a wave per row 89 / 89 / 80).
        if (GUARD) {
            for (uint32_t e = grp; e < cnt; e += ng)
                if (skey[e] == SA_SLOW)
                    add_row_exact<GUARD, W>(dst, rb, idx, src, c0 + spos[e], rg, lir, G, acc);
            __syncthreads();
        }
    }
    if (GUARD && logon) end_faults(acc, log, fin);
}

// ================================================================ sorted path
constexpr int SRT_BLOCK = 256;
constexpr uint32_t SRT_TILE = 4096;   // keys per histogram / scatter tile (16 per thread)
constexpr uint32_t SRT_TB = 1024;      // threads of the histogram and scatter workgroups
constexpr uint32_t SRT_SENT = 0xFFFFFFFFu;
constexpr uint32_t RED_TILE = 128;    // most sorted entries per tile of the reduce
// ctl[p] (p < 4): pass p was skipped (one digit value only); ctl[4 + p]: the buffer pass p reads
// (ctl[4 + npasses]: the buffer holding the sorted result, which the reduce reads)
constexpr int CTL_WORDS = 16;

struct SortBufs {
    uint32_t* keys[2];
    uint32_t* vals[2];
    uint32_t* hist;  // [257 * ntiles], scanned in place (row 256, first pass: guard-failing rows)
    uint32_t* ctl;   // [CTL_WORDS]
    uint32_t* dstart;  // [256]: the current pass's digit totals; [256]: all guard-failing rows
};

static inline uint64_t srt_ntiles(uint64_t n) { return (n + SRT_TILE - 1) / SRT_TILE; }

size_t scatter_add_scratch_bytes(uint64_t n) {
    const uint64_t a = ((n * 4 + 255) / 256) * 256;
    return 4 * a + srt_ntiles(n) * 257 * 4 + 256 + 1280;
}

static SortBufs sort_bufs(void* scratch, uint64_t n) {
    const uint64_t a = ((n * 4 + 255) / 256) * 256;
    uint8_t* p = static_cast<uint8_t*>(scratch);
    SortBufs b;
    b.keys[0] = reinterpret_cast<uint32_t*>(p);
    b.keys[1] = reinterpret_cast<uint32_t*>(p + a);
    b.vals[0] = reinterpret_cast<uint32_t*>(p + 2 * a);
    b.vals[1] = reinterpret_cast<uint32_t*>(p + 3 * a);
    b.hist = reinterpret_cast<uint32_t*>(p + 4 * a);
    b.ctl = reinterpret_cast<uint32_t*>(p + 4 * a + srt_ntiles(n) * 257 * 4);
    b.dstart = reinterpret_cast<uint32_t*>(p + 4 * a + srt_ntiles(n) * 257 * 4 + 256);
    return b;
}

// Keys: guarded rows that pass the fast test get (idx - rlo); the others the sentinel. The
// unguarded twin keys every row by idx + 2^31 (its indices must lie in [-2^31, 2^31 - 1)). One
// workgroup per tile of SRT_TILE rows, which also counts the tile's digits of the first pass, so
// the sort's first histogram needs no pass over the keys of its own.
template <bool GUARD>
__global__ __launch_bounds__(SRT_TB) void k_srt_keys(const int64_t* __restrict__ idx, uint64_t n,
                                                     RowsGuard rg, SortBufs b) {
    __shared__ uint32_t h[257];
    const uint32_t tid = threadIdx.x;
    if (blockIdx.x == 0 && tid < CTL_WORDS) b.ctl[tid] = 0;  // every pass starts from buffer 0
    if (tid < 257) h[tid] = 0;
    __syncthreads();
    const uint64_t t0 = (uint64_t)blockIdx.x * SRT_TILE;
#pragma unroll
    for (uint32_t r = 0; r < SRT_TILE / SRT_TB; ++r) {
        const uint64_t i = t0 + r * SRT_TB + tid;
        if (i < n) {
            uint32_t key = SRT_SENT;
            if (GUARD) {
                const int64_t x = i < rg.nfast ? idx[i] : 0;
                const bool fast = i < rg.nfast && rg.g.rlo <= x && x <= rg.g.rhi;
                if (fast) key = (uint32_t)((uint64_t)x - (uint64_t)rg.g.rlo);
                else atomicAdd(&h[256], 1u);
            } else {
                key = (uint32_t)((uint64_t)idx[i] + 0x80000000ull);
            }
            b.keys[0][i] = key;
            b.vals[0][i] = (uint32_t)i;
            atomicAdd(&h[key & 255u], 1u);
        }
    }
    __syncthreads();
    if (tid < 257) b.hist[(uint64_t)tid * gridDim.x + blockIdx.x] = h[tid];
}

// Digit histogram of one pass per tile of SRT_TILE keys, stored digit-major (hist[d * ntiles + t]).
__global__ __launch_bounds__(SRT_TB) void k_srt_hist(SortBufs b, uint64_t n, uint32_t pass) {
    __shared__ uint32_t h[256];
    const uint32_t tid = threadIdx.x, shift = 8 * pass;
    const uint32_t* keys = b.keys[b.ctl[4 + pass]];
    if (tid < 256) h[tid] = 0;
    __syncthreads();
    const uint64_t t0 = (uint64_t)blockIdx.x * SRT_TILE;
    uint32_t k[SRT_TILE / SRT_TB];
#pragma unroll
    for (uint32_t r = 0; r < SRT_TILE / SRT_TB; ++r) {
        const uint64_t i = t0 + r * SRT_TB + tid;
        k[r] = i < n ? keys[i] : 0u;
    }
#pragma unroll
    for (uint32_t r = 0; r < SRT_TILE / SRT_TB; ++r)
        if (t0 + r * SRT_TB + tid < n) atomicAdd(&h[(k[r] >> shift) & 255u], 1u);
    __syncthreads();
    if (tid < 256) b.hist[(uint64_t)tid * gridDim.x + blockIdx.x] = h[tid];
}

// Offsets of a pass. k_srt_scan_rows: one workgroup per digit turns the digit's per-tile counts
// into exclusive prefixes and records the digit's total; the scatter's workgroups then turn the
// 256 totals into each digit's first output position themselves.
template <uint32_t NT>
__device__ inline uint32_t block_scan(uint32_t v, uint32_t* wsum, uint32_t& total) {
    const uint32_t tid = threadIdx.x, lane = tid & 63u, wv = tid >> 6;
    uint32_t inc = v;
    for (int o = 1; o < 64; o <<= 1) {
        const uint32_t y = __shfl_up(inc, o, 64);
        if (lane >= (uint32_t)o) inc += y;
    }
    if (lane == 63) wsum[wv] = inc;
    __syncthreads();
    uint32_t before = 0;
    total = 0;
    for (uint32_t k = 0; k < NT / 64; ++k) {
        if (k < wv) before += wsum[k];
        total += wsum[k];
    }
    __syncthreads();
    return before + inc - v;
}

__global__ __launch_bounds__(SRT_BLOCK) void k_srt_scan_rows(SortBufs b, uint32_t ntiles) {
    __shared__ uint32_t wsum[SRT_BLOCK / 64];
    uint32_t* row = b.hist + (uint64_t)blockIdx.x * ntiles;
    uint32_t carry = 0;
    for (uint32_t t0 = 0; t0 < ntiles; t0 += SRT_BLOCK) {
        const uint32_t t = t0 + threadIdx.x;
        const uint32_t v = t < ntiles ? row[t] : 0u;
        uint32_t total;
        const uint32_t ex = block_scan<SRT_BLOCK>(v, wsum, total);
        if (t < ntiles) row[t] = carry + ex;
        carry += total;
    }
    if (threadIdx.x == 0) b.dstart[blockIdx.x] = carry;
}

// Stable scatter of one pass over a tile of SRT_TILE keys. The workgroup first turns the 256 digit
// totals into each digit's first output position (a pass whose digit is the same for all n keys is
// skipped; workgroup 0 records that, and which buffer the next pass reads). Each wave then ranks
// its SRT_TILE / 16 consecutive keys by digit in rounds of 64: wave ballots rank equal digits by
// lane, and a per-wave running count per digit carries the order from round to round (a wave's
// LDS reads and writes take effect in program order, so no barrier is needed between rounds).
// The tile's keys are regrouped by digit in LDS, in position order within a digit, and each
// digit's group is written to its place in the output as one contiguous run.
__global__ __launch_bounds__(SRT_TB) void k_srt_scatter(SortBufs b, uint64_t n, uint32_t pass) {
    constexpr uint32_t NW = SRT_TB / 64;
    constexpr uint32_t R = SRT_TILE / SRT_TB;  // rounds per wave
    __shared__ uint32_t wc[NW][256];  // keys per wave and digit, then each wave's offset in the digit
    __shared__ uint32_t lstart[256];  // first slot of each digit in the regrouped tile
    __shared__ uint32_t gstart[256];  // output position of the tile's first key of each digit
    __shared__ uint32_t sk[SRT_TILE], sv[SRT_TILE];
    __shared__ uint32_t wsum[NW];
    __shared__ uint32_t skip;
    const uint32_t tid = threadIdx.x, lane = tid & 63u, wv = tid >> 6, shift = 8 * pass;
    const uint32_t src = b.ctl[4 + pass];
    if (tid == 0) skip = 0;
    const uint32_t tot = tid < 256 ? b.dstart[tid] : 0u;
    __syncthreads();
    if (tid < 256 && (uint64_t)tot == n) skip = 1;
    uint32_t all;
    const uint32_t dfirst = block_scan<SRT_TB>(tot, wsum, all);
    if (blockIdx.x == 0 && tid == 0) {
        b.ctl[pass] = skip;
        b.ctl[4 + pass + 1] = skip ? src : 1u - src;
    }
    if (skip) return;
    const uint32_t* kin = b.keys[src];
    const uint32_t* vin = b.vals[src];
    uint32_t* kout = b.keys[1u - src];
    uint32_t* vout = b.vals[1u - src];
    if (tid < 256) {
#pragma unroll
        for (uint32_t w = 0; w < NW; ++w) wc[w][tid] = 0;
        gstart[tid] = dfirst + b.hist[(uint64_t)tid * gridDim.x + blockIdx.x];
    }
    __syncthreads();
    const uint64_t t0 = (uint64_t)blockIdx.x * SRT_TILE;
    const uint64_t w0 = t0 + (uint64_t)wv * (SRT_TILE / NW);
    const uint64_t below = lane ? (~0ull >> (64 - lane)) : 0ull;
    uint32_t key[R], val[R], pre[R];
#pragma unroll
    for (uint32_t r = 0; r < R; ++r) {
        const uint64_t i = w0 + r * 64 + lane;
        key[r] = i < n ? kin[i] : 0u;
        val[r] = i < n ? vin[i] : 0u;
    }
#pragma unroll
    for (uint32_t r = 0; r < R; ++r) {
        const bool valid = w0 + r * 64 + lane < n;
        const uint32_t d = (key[r] >> shift) & 255u;
        uint64_t match = __ballot(valid);
#pragma unroll
        for (int bit = 0; bit < 8; ++bit) {
            const uint64_t bb = __ballot((d >> bit) & 1u);
            match &= ((d >> bit) & 1u) ? bb : ~bb;
        }
        const uint32_t rank = (uint32_t)__popcll(match & below);
        pre[r] = wc[wv][d] + rank;
        if (valid && rank == 0) wc[wv][d] = pre[r] + (uint32_t)__popcll(match);
    }
    __syncthreads();
    // thread tid < 256 owns digit tid: the tile's count, and each wave's offset inside the digit
    uint32_t cnt = 0;
    if (tid < 256) {
#pragma unroll
        for (uint32_t w = 0; w < NW; ++w) {
            const uint32_t c = wc[w][tid];
            wc[w][tid] = cnt;
            cnt += c;
        }
    }
    const uint32_t lfirst = block_scan<SRT_TB>(cnt, wsum, all);
    if (tid < 256) lstart[tid] = lfirst;
    __syncthreads();
#pragma unroll
    for (uint32_t r = 0; r < R; ++r) {
        if (w0 + r * 64 + lane < n) {
            const uint32_t d = (key[r] >> shift) & 255u;
            const uint32_t slot = lstart[d] + wc[wv][d] + pre[r];
            sk[slot] = key[r];
            sv[slot] = val[r];
        }
    }
    __syncthreads();
    const uint32_t m = (uint32_t)(n - t0 < SRT_TILE ? n - t0 : SRT_TILE);
    for (uint32_t q = tid; q < m; q += SRT_TB) {
        const uint32_t k = sk[q];
        const uint32_t d = (k >> shift) & 255u;
        const uint32_t pos = gstart[d] + (q - lstart[d]);
        kout[pos] = k;
        vout[pos] = sv[q];
    }
}

template <int W, int EPL>
struct RowVec {
    typename FloatOf<W>::F v[EPL];
};

// NT: a row read once (a source row of the sum): non-temporal, so it does not push the
// destination rows, which are read, summed and written back, out of the caches.
template <int W, int EPL, bool NT = false>
__device__ __forceinline__ RowVec<W, EPL> load_row(const uint8_t* src, uint64_t rb, uint32_t row,
                                                   uint64_t col0) {
    using F = typename FloatOf<W>::F;
    typedef F fv __attribute__((ext_vector_type(EPL), aligned(W)));
    RowVec<W, EPL> r;
    const F* sp = reinterpret_cast<const F*>(src + (uint64_t)row * rb) + col0;
    const fv* vp = reinterpret_cast<const fv*>(sp);
    const fv v = NT ? __builtin_nontemporal_load(vp) : *vp;
#pragma unroll
    for (int q = 0; q < EPL; ++q) r.v[q] = v[q];
    return r;
}

// End of a run: an owned destination row gets (its value loaded when the run started + the
// run's sum) stored back; a shared one gets atomic adds. The first `skip` columns are another lane's.
template <int W, int EPL>
__device__ __forceinline__ void srt_flush(uint8_t* dst, uint64_t rb, int64_t row, uint64_t col0,
                                          uint32_t skip, bool owned, const RowVec<W, EPL>& old,
                                          const typename FloatOf<W>::F (&acc)[EPL]) {
    using F = typename FloatOf<W>::F;
    typedef F fv __attribute__((ext_vector_type(EPL), aligned(W)));
    F* d = reinterpret_cast<F*>(dst + (uint64_t)row * rb) + col0;
    if (owned) {
        fv v;
#pragma unroll
        for (int q = 0; q < EPL; ++q) v[q] = old.v[q] + acc[q];
        if (EPL == 1 || skip == 0) {
            *reinterpret_cast<fv*>(d) = v;
        } else {
#pragma unroll
            for (int q = 1; q < EPL; ++q)
                if ((uint32_t)q >= skip) d[q] = v[q];
        }
    } else {
#pragma unroll
        for (int q = 0; q < EPL; ++q)
            if (EPL == 1 || (uint32_t)q >= skip) unsafeAtomicAdd(d + q, acc[q]);
    }
}

// A group of 2^glog2 lanes walks a tile of `tile` sorted entries with RED_U rows in flight: the source
// rows of the next RED_U entries are loaded together with the destination row of every run that
// starts among them, then the rows are summed in order. A run that the tile owns ends with a plain
// store of (destination + sum). A run that spans tiles of the workgroup is put together in LDS by
// the group in whose tile it ends, and ends there the same way; a run shared with a neighbouring
// workgroup ends with one atomic add per element and workgroup. ROW_WAVE: rows of at least 64 chunks,
// a wave per row, whose keys and positions are held one per lane and read out wave-uniformly.
// Bound by the random row reads; with one atomic add per tile instead of per workgroup the atomics
// on the hottest rows, about 100 ns each one after another, set the time instead (1 KiB rows, 2^20 of
// them: 298 us with tiles of 256, more with shorter ones; now 265 us with 128, 270 with 64, 280 with 256).
constexpr int RED_U = 8;
// zero_dst: the destination rows are +0.0 before the call (the caller's promise), so the rows are
// not read: an owned run stores (+0.0 + sum), exactly what the read-modify-write would.
template <bool GUARD, int W, int EPL, bool ROW_WAVE>
__global__ __launch_bounds__(256, ROW_WAVE ? 4 : 3) void k_srt_reduce(uint8_t* dst, uint64_t rb,
                                                       const uint8_t* __restrict__ src, uint64_t n,
                                                       SortBufs b, uint32_t npasses, int64_t rlo,
                                                       uint32_t zero_dst, uint32_t tile,
                                                       uint32_t glog2) {
    using F = typename FloatOf<W>::F;
    __shared__ F part[EPL][256];  // sum of each tile's last run, if the next tile goes on with it
    __shared__ uint32_t whole[32];  // the tile is one run that goes on from the previous tile
    const uint32_t tid = threadIdx.x, lane = tid & 63u;
    const uint32_t gl = ROW_WAVE ? 6u : glog2;
    const uint32_t lir = tid & ((1u << gl) - 1), grp = tid >> gl, ng = 256u >> gl;
    const uint32_t buf = b.ctl[4 + npasses];
    const uint32_t* __restrict__ keys = b.keys[buf];
    const uint32_t* __restrict__ vals = b.vals[buf];
    const uint64_t D = rb / W;
    const int64_t base = GUARD ? rlo : -(int64_t)0x80000000ll;
    const uint64_t span = (uint64_t)tile * ng;  // entries per workgroup
    for (uint64_t b0 = (uint64_t)blockIdx.x * span; b0 < n; b0 += (uint64_t)gridDim.x * span) {
        if (keys[b0] == SRT_SENT) break;
        uint64_t e0 = b0 + (uint64_t)grp * tile;
        if (ROW_WAVE) e0 = uniform_u64(e0);
        const uint64_t e1 = e0 + tile < n ? e0 + tile : n;
        uint32_t k0 = e0 < n ? keys[e0] : SRT_SENT;
        if (ROW_WAVE) k0 = (uint32_t)__builtin_amdgcn_readfirstlane((int)k0);
        const bool some = k0 != SRT_SENT;
        const uint32_t klast = some ? keys[e1 - 1] : SRT_SENT;
        // does the tile's first run go on from the previous tile, its last run into the next?
        const bool head_on = some && e0 > 0 && keys[e0 - 1] == k0;
        const bool tail_on = some && e1 < n && klast != SRT_SENT && keys[e1] == klast;
        const bool from_prev = head_on && grp > 0, to_next = tail_on && grp + 1 < ng;
        if (lir == 0) whole[grp] = head_on && k0 == klast;
        for (uint64_t cb = 0; cb < D; cb += (uint64_t)EPL << gl) {
            // a row that ends inside a vector: its last lane's vector ends with the row
            const uint64_t c0 = cb + (uint64_t)lir * EPL, col0 = EPL == 1 || c0 + EPL <= D ? c0 : D - EPL;
            const uint32_t skip = (uint32_t)(c0 - col0);
            const bool on = some && c0 < D;
            F acc[EPL], head[EPL];  // head: the end of a run that earlier tiles began
#pragma unroll
            for (int q = 0; q < EPL; ++q) acc[q] = (F)-0.0;
            uint32_t cur = k0;
            bool first = true, ends_here = false;
            RowVec<W, EPL> dcur;
#pragma unroll
            for (int q = 0; q < EPL; ++q) dcur.v[q] = (F)0.0;
            if (on && !head_on && !zero_dst)
                dcur = load_row<W, EPL>(dst + (uint64_t)(base + (int64_t)k0) * rb, rb, 0, col0);
            uint32_t tk = 0, tv = 0;
            if (ROW_WAVE ? some : on) {
                for (uint64_t e = e0; e < e1; e += RED_U) {
                    uint32_t kk[RED_U], vv[RED_U];
                    RowVec<W, EPL> rv[RED_U], dv[RED_U];
                    if (ROW_WAVE) {
                        const uint32_t l = (uint32_t)(e - e0) & 63u;
                        if (l == 0) {
                            tk = e + lane < e1 ? keys[e + lane] : SRT_SENT;
                            tv = e + lane < e1 ? vals[e + lane] : 0u;
                        }
#pragma unroll
                        for (int u = 0; u < RED_U; ++u) {
                            kk[u] = (uint32_t)__builtin_amdgcn_readlane((int)tk, (int)(l + u));
                            vv[u] = (uint32_t)__builtin_amdgcn_readlane((int)tv, (int)(l + u));
                        }
                        if (kk[0] == SRT_SENT) break;
                    } else {
#pragma unroll
                        for (int u = 0; u < RED_U; ++u) {
                            const uint64_t x = e + u < e1 ? e + u : e1 - 1;
                            kk[u] = e + u < e1 ? keys[x] : SRT_SENT;
                            vv[u] = vals[x];
                        }
                    }
#pragma unroll
                    for (int u = 0; u < RED_U; ++u) {
                        if (kk[u] != SRT_SENT && on) {
                            rv[u] = load_row<W, EPL, true>(src, rb, vv[u], col0);
                            if (kk[u] != (u == 0 ? cur : kk[u - 1])) {
                                if (zero_dst) {
#pragma unroll
                                    for (int q = 0; q < EPL; ++q) dv[u].v[q] = (F)0.0;
                                } else {
                                    dv[u] = load_row<W, EPL>(dst + (uint64_t)(base + (int64_t)kk[u]) * rb,
                                                             rb, 0, col0);
                                }
                            }
                        }
                    }
#pragma unroll
                    for (int u = 0; u < RED_U; ++u) {
                        if (kk[u] != SRT_SENT) {
                            if (kk[u] != cur) {
                                if (first && from_prev) {
                                    ends_here = true;
#pragma unroll
                                    for (int q = 0; q < EPL; ++q) head[q] = acc[q];
                                } else if (on) {
                                    srt_flush<W, EPL>(dst, rb, base + (int64_t)cur, col0, skip,
                                                      !(first && head_on), dcur, acc);
                                }
#pragma unroll
                                for (int q = 0; q < EPL; ++q) acc[q] = (F)-0.0;
                                cur = kk[u];
                                dcur = dv[u];
                                first = false;
                            }
                            if (on) {
#pragma unroll
                                for (int q = 0; q < EPL; ++q) acc[q] += rv[u].v[q];
                            }
                        }
                    }
                }
            }
            // the last run: its sum goes to the next tile's group, joins an earlier tile's, or is flushed
            const bool last_on = tail_on && cur == klast;
            bool tail_out = false;  // the run put together here goes on in the next workgroup
            if (on) {
                if (last_on && to_next) {
#pragma unroll
                    for (int q = 0; q < EPL; ++q) part[q][tid] = acc[q];
                } else if (first && from_prev) {
                    ends_here = true;
                    tail_out = last_on;
#pragma unroll
                    for (int q = 0; q < EPL; ++q) head[q] = acc[q];
                } else {
                    srt_flush<W, EPL>(dst, rb, base + (int64_t)cur, col0, skip,
                                      !((first && head_on) || last_on), dcur, acc);
                }
            }
            __syncthreads();
            if (on && ends_here) {
                uint32_t p = grp - 1;  // the tile in which the run begins, or the workgroup's first
                while (p > 0 && whole[p]) --p;
                const bool owned = !tail_out && !whole[p];  // whole[0]: an earlier workgroup's run
                RowVec<W, EPL> old;
#pragma unroll
                for (int q = 0; q < EPL; ++q) old.v[q] = (F)0.0;
                if (owned && !zero_dst)
                    old = load_row<W, EPL>(dst + (uint64_t)(base + (int64_t)k0) * rb, rb, 0, col0);
                F run[EPL];
#pragma unroll
                for (int q = 0; q < EPL; ++q) run[q] = (F)-0.0;
                for (; p < grp; ++p)
#pragma unroll
                    for (int q = 0; q < EPL; ++q) run[q] += part[q][(p << gl) + lir];
#pragma unroll
                for (int q = 0; q < EPL; ++q) run[q] += head[q];
                srt_flush<W, EPL>(dst, rb, base + (int64_t)k0, col0, skip, owned, old, run);
            }
            __syncthreads();
        }
    }
}

// Rows that failed the fast test: every element checked exactly, atomics for the allowed ones. They
// sorted last (largest key), and the first scan counted them. In a kernel of their own behind the
// reduce, whose owned rows take plain stores. All of the sorted path's denials come from these rows,
// so the last workgroup to finish also records them.
template <int W>
__global__ __launch_bounds__(256) void k_srt_slow(DevLog* log, uint8_t* dst, uint64_t rb,
                                                  const int64_t* idx, const uint8_t* src,
                                                  uint64_t n, RowsGuard rg, SortBufs b,
                                                  uint32_t npasses, int logon, FinishArgs fin) {
    const uint32_t slow = b.dstart[256];
    if (slow == 0) return;
    const uint32_t* vals = b.vals[b.ctl[4 + npasses]];
    FaultAcc acc;
    // four rows at a time, so that fewer waves fold their denials into the log's one cache line
    const uint64_t wave = blockIdx.x * 4u + (threadIdx.x >> 6), step = (uint64_t)gridDim.x * 16;
    for (uint64_t e0 = n - slow + wave * 4; e0 < n; e0 += step)
        for (uint64_t e = e0; e < n && e < e0 + 4; ++e)
            add_row_exact<true, W>(dst, rb, idx, src, vals[e], rg, threadIdx.x & 63u, 64, acc);
    if (logon) end_faults(acc, log, fin);
}

// Lanes per row: enough to cover its chunks, at most a wave.
static uint32_t row_lanes_log2(uint64_t nch) {
    uint32_t l = 0;
    while (l < 6 && (1ull << l) < nch) ++l;
    return l;
}

template <bool G, int W, int EPL>
static void reduce_sorted(void* dst, uint64_t rb, const void* src, uint64_t n, const RowsGuard& rg,
                          uint32_t npasses, const SortBufs& b, const DevInfo& d, hipStream_t s,
                          bool zero_dst) {
    // at least 8 lanes a group: at most 32 tiles of a workgroup are put together one after another
    const uint32_t rl = row_lanes_log2((rb / W + EPL - 1) / EPL), gl = rl < 3 ? 3 : rl;
    // short tiles until four waves for every SIMD of the chip remain, then longer ones
    uint32_t tile = gl == 6 ? 64 : 32;
    while (tile < RED_TILE && (n >> (6 - gl)) / (2 * tile) >= (uint64_t)d.num_cu * 16) tile *= 2;
    const uint64_t span = (uint64_t)tile * (256 >> gl);
    const uint64_t blocks = (n + span - 1) / span, cap = 1ull << 22;
    const dim3 grid((uint32_t)(blocks < cap ? blocks : cap)), block(256);
    if (gl == 6)
        hipLaunchKernelGGL((k_srt_reduce<G, W, EPL, true>), grid, block, 0, s, (uint8_t*)dst, rb,
                           (const uint8_t*)src, n, b, npasses, rg.g.rlo, (uint32_t)zero_dst, tile, gl);
    else
        hipLaunchKernelGGL((k_srt_reduce<G, W, EPL, false>), grid, block, 0, s, (uint8_t*)dst, rb,
                           (const uint8_t*)src, n, b, npasses, rg.g.rlo, (uint32_t)zero_dst, tile, gl);
}

// A scatter-add's launch, and what its denials need.
struct AddCall {
    GuardTab t;
    DevLog* log;
    uint8_t* dst;
    uint64_t rb;
    const int64_t* idx;
    const uint8_t* src;
    uint64_t n;
    RowsGuard rg;
    FaultSite site;
    unsigned long long seq;
    int logon;
    bool finish;
    DevInfo d;
    hipStream_t s;
};

template <bool G, int W>
static hipError_t scatter_add_sorted(const AddCall& c, uint32_t npasses, void* scratch, bool zero_dst) {
    const SortBufs b = sort_bufs(scratch, c.n);
    const uint32_t ntiles = (uint32_t)srt_ntiles(c.n);
    // the key pass also writes the first pass's per-tile histograms
    hipLaunchKernelGGL((k_srt_keys<G>), dim3(ntiles), dim3(SRT_TB), 0, c.s, c.idx, c.n, c.rg, b);
    for (uint32_t p = 0; p < npasses; ++p) {
        if (p > 0) hipLaunchKernelGGL(k_srt_hist, dim3(ntiles), dim3(SRT_TB), 0, c.s, b, c.n, p);
        hipLaunchKernelGGL(k_srt_scan_rows, dim3(p == 0 ? 257 : 256), dim3(SRT_BLOCK), 0, c.s, b, ntiles);
        hipLaunchKernelGGL(k_srt_scatter, dim3(ntiles), dim3(SRT_TB), 0, c.s, b, c.n, p);
    }
    const uint64_t D = c.rb / W;
    const auto reduce = [&](auto epl) {
        reduce_sorted<G, W, decltype(epl)::value>(c.dst, c.rb, c.src, c.n, c.rg, npasses, b, c.d, c.s, zero_dst);
    };
    // Elements per lane: so many that 33-64 lanes cover a row, if any number does (a wave per row, keys
    // and guard in scalar registers; with the whole vectors that alignment allowed before, or single
    // elements, 2^19 rows of 64 floats 135 us against 116, of 65 164 / 131, of 128 174 / 142, 48 doubles
    // 157 / 127); below that vectors from half a wave's worth on (17 floats 127 / 106), above it whole ones
    // (129 floats 212 / 165, 65 doubles 190 / 156).
    if (D <= 16 || (D > 32 && D <= 64)) reduce(std::integral_constant<int, 1>{});
    else if (W == 8 || (D > 64 && D <= 128)) reduce(std::integral_constant<int, 2>{});
    else reduce(std::integral_constant<int, 16 / W>{});
    if constexpr (G) {
        const uint64_t sb = (c.n + 255) / 256, cap = (uint64_t)c.d.num_cu * 4;
        const uint32_t grid = (uint32_t)(sb < cap ? sb : cap);
        const bool wanted = c.logon && c.finish;
        const FinishArgs fin = finish_args(c.t, c.site, c.seq, grid, wanted, c.s);
        hipLaunchKernelGGL((k_srt_slow<W>), dim3(grid), dim3(256), 0, c.s, c.log, c.dst, c.rb, c.idx, c.src,
                           c.n, c.rg, b, npasses, c.logon, fin);
        if (wanted && !fin.fused) return launch_fault_finish(c.t, c.log, c.site, c.seq, c.s);
    }
    return hipGetLastError();
}

template <bool G, int W, int EPL, int CH, int TB>
static hipError_t scatter_add_chunks(const AddCall& c, uint32_t gl) {
    const uint64_t chunks = (c.n + CH - 1) / CH, cap = (uint64_t)c.d.num_cu * 8;
    const uint32_t grid = (uint32_t)(chunks < cap ? chunks : cap);
    const auto launch = [&](const auto& fin) {
        hipLaunchKernelGGL((k_scatter_add<G, W, EPL, CH, TB>), dim3(grid), dim3(TB), 0, c.s, c.log, c.dst,
                           c.rb, c.idx, c.src, c.n, c.rg, c.logon, gl, fin);
    };
    if constexpr (G) {
        const bool wanted = c.logon && c.finish;
        const FinishArgs fin = finish_args(c.t, c.site, c.seq, grid, wanted, c.s);
        launch(fin);
        if (wanted && !fin.fused) return launch_fault_finish(c.t, c.log, c.site, c.seq, c.s);
    } else {
        launch(NoFinish{});
    }
    return hipGetLastError();
}

template <bool G, int W>
static hipError_t scatter_add_w(const AddCall& c) {
    constexpr int EPL = W == 4 ? 4 : 2;
    const uint32_t gl = row_lanes_log2((c.rb / W + EPL - 1) / EPL);
    uint64_t ch = 64;
    while (ch < 1024 && c.n > SA_CHUNKS * ch) ch *= 2;
    switch (ch) {
        case 64: return scatter_add_chunks<G, W, EPL, 64, 256>(c, gl);
        case 128: return scatter_add_chunks<G, W, EPL, 128, 256>(c, gl);
        case 256: return scatter_add_chunks<G, W, EPL, 256, 1024>(c, gl);
        case 512: return scatter_add_chunks<G, W, EPL, 512, 1024>(c, gl);
        default: return scatter_add_chunks<G, W, EPL, 1024, 1024>(c, gl);
    }
}

hipError_t launch_scatter_add(bool guard, const GuardTab& t, DevLog* log, const Bind* binds,
                              void* dst, uint64_t rb, const int64_t* idx, const void* src,
                              uint64_t n, uint32_t w, unsigned long long seq, int logon,
                              void* scratch, const DevInfo& d, hipStream_t s, bool finish,
                              bool zero_dst) {
    if (n == 0) return hipSuccess;
    AddCall c{t, log, static_cast<uint8_t*>(dst), rb, idx, static_cast<const uint8_t*>(src), n,
              guard ? rows_guard(binds[0], binds[1], binds[2], (uint64_t)idx, (uint64_t)src, (uint64_t)dst,
                                 n, rb, w)
                    : rows_open(n, rb, w),
              FaultSite{}, seq, logon, finish, d, s};
    if (guard) c.site = rows_fault_site(5 /*OP_SCATTER_ADD*/, w, 2, rb, c.rg.ki, idx, src, dst);
    // sorted path: 32-bit keys (guarded: the destination's row interval minus the sentinel;
    // unguarded: idx + 2^31), positions below 2^32
    uint32_t npasses = 0;
    bool sorted = scratch != nullptr && scatter_add_sorts(n, rb) && n < (1ull << 32);
    if (sorted && guard) {
        if (!c.rg.g.bound || c.rg.g.rhi < c.rg.g.rlo) {
            npasses = 1;  // no fast rows: every key is the sentinel, the sort is trivial
        } else {
            const uint64_t span = (uint64_t)c.rg.g.rhi - (uint64_t)c.rg.g.rlo;
            if (span >= SRT_SENT) sorted = false;
            // enough bits for span + 1, so that no key equals the sentinel in the sorted bits
            // (the largest key of a 2^16-row table is all ones in 16 bits)
            uint32_t bits = 0;
            while (bits < 32 && ((span + 1) >> bits)) ++bits;
            npasses = (bits + 7) / 8;
            if (npasses == 0) npasses = 1;
        }
    } else if (sorted) {
        npasses = 4;
    }
    if (sorted) {
        if (guard) return w == 4 ? scatter_add_sorted<true, 4>(c, npasses, scratch, zero_dst)
                                 : scatter_add_sorted<true, 8>(c, npasses, scratch, zero_dst);
        return w == 4 ? scatter_add_sorted<false, 4>(c, npasses, scratch, zero_dst)
                      : scatter_add_sorted<false, 8>(c, npasses, scratch, zero_dst);
    }
    if (guard) return w == 4 ? scatter_add_w<true, 4>(c) : scatter_add_w<true, 8>(c);
    return w == 4 ? scatter_add_w<false, 4>(c) : scatter_add_w<false, 8>(c);
}

}  // namespace agile
