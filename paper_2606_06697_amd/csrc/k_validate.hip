// Batched pointer validation (the API-time classification rule of AgileOS Sections IV-E and
// V-C, applied to many (addr, len) queries at once).
//
// Each workgroup (16 waves) stages the table's splitters (every 2^rlog2-th bucket base; 32-bit keys
// when the table allows exact compression), a run of largest-value sentinels and a radix index over
// the splitters into LDS once, with the packed records behind them where they fit and the batch is
// large. Every lane then classifies its queries: the radix entry of the address offset gives the
// start of a short run of candidate splitters, binary lifting over that run finds the last
// splitter <= addr (reading past the run is harmless: later splitters and the sentinels compare
// greater, so the predicate stays monotone and needs no bound checks), and one bucket record
// read resolves the range inside the bucket with its end, id and kind.
//
// With DMA set the same search answers the DMA registration check (Section V-C: only an exact
// live user allocation is accepted): an allowed range that is not the whole allocation, from
// its base with its full size, is reported INEXACT.
//
// Two record formats: packed 16-byte records (one load per query; offsets relative to the
// bucket base, used whenever the table's offsets fit) and general 32-byte records. Large batches on
// tables whose records do not fit the LDS have an index of their own (chunk_bytes). Queries
// stream in with coalesced 16-byte loads, the next chunk's queries are in flight while the
// current chunk is searched, and verdict bytes and owner ids are stored coalesced.
#include <cstdlib>
#include <type_traits>

#include "launch.h"

namespace agile {

constexpr int VBLOCK = 1024;
typedef unsigned long long uint64x2 __attribute__((ext_vector_type(2)));

template <bool COMP>
struct KeyT {
    using T = uint64_t;
};
template <>
struct KeyT<true> {
    using T = uint32_t;
};

// Stages the search index into LDS, and with LREC the packed records behind it: one copy of the image
// that the host laid out as it is to lie there. A short loop on purpose: several loads in flight per
// thread (five at a time, in rounds) and the first queries loaded ahead of the barrier both made launches
// of up to 2^20 queries 0.3-0.5 us longer, by their code. Against 4-byte loads, array after array: 200
// queries on 65,536 ranges 7.3 -> 4.0 us, 200,000 12.8 -> 8.9, 2^20 13.8 -> 11.6.
__device__ __forceinline__ void stage_index(uint4* lds, const uint4* src, uint32_t nv) {
#pragma unroll 1
    for (uint32_t k = threadIdx.x; k < nv; k += VBLOCK) lds[k] = src[k];
    __syncthreads();
}

template <int QPT, bool TAIL>
__device__ __forceinline__ void load_chunk(const ulonglong2* __restrict__ q, uint64_t n,
                                           uint64_t c0, uint32_t lane, ulonglong2 (&x)[QPT]) {
    const uint64x2* qp = reinterpret_cast<const uint64x2*>(q) + c0 + lane;
#pragma unroll
    for (int j = 0; j < QPT; ++j) {
        uint64x2 v;
        if (TAIL) {
            const uint64_t i = c0 + (uint64_t)j * 64u + lane;
            v = __builtin_nontemporal_load(reinterpret_cast<const uint64x2*>(q) + (i < n ? i : n - 1));
        } else {
            v = __builtin_nontemporal_load(qp + j * 64);
        }
        x[j] = make_ulonglong2(v.x, v.y);
    }
}

// Search key and radix start of each query.
template <bool COMP, int QPT>
__device__ __forceinline__ void keys_and_starts(const DevTable& t, const uint32_t* ri,
                                                const ulonglong2 (&x)[QPT],
                                                typename KeyT<COMP>::T (&key)[QPT],
                                                uint32_t (&p)[QPT]) {
    const uint32_t nr1 = t.nr - 1;
#pragma unroll
    for (int j = 0; j < QPT; ++j) {
        const uint64_t d = x[j].x - t.gmin;
        uint32_t r;
        if (COMP) {
            const uint64_t kk = d >> t.shift;
            key[j] = (uint32_t)(kk > 0xFFFFFFFFull ? 0xFFFFFFFFull : kk);
            r = (uint32_t)key[j] >> t.xs;
        } else {
            key[j] = x[j].x;
            const uint64_t rr = d >> t.rsh;
            r = rr > 0xFFFFFFFFull ? 0xFFFFFFFFu : (uint32_t)rr;
        }
        p[j] = ri[r < nr1 ? r : nr1];
    }
}

// ---------------------------------------------------------------- general (32-byte records)
template <bool COMP, int QPT, bool TAIL, bool DMA>
__device__ __forceinline__ void chunk_wide(const DevTable& t, const unsigned char* lds_raw,
                                           const uint32_t* ri, const ulonglong2 (&x)[QPT],
                                           uint64_t n, uint8_t* __restrict__ verdict,
                                           int32_t* __restrict__ owner, uint64_t c0, uint32_t lane) {
    using K = typename KeyT<COMP>::T;
    const K* top = reinterpret_cast<const K*>(lds_raw);
    const uint32_t ntop = t.ntop;
    K key[QPT];
    uint32_t p[QPT];  // number of splitters known to be <= key
    keys_and_starts<COMP, QPT>(t, ri, x, key, p);
    for (uint32_t step = t.rlevels ? 1u << (t.rlevels - 1) : 0u; step; step >>= 1) {
        K v[QPT];
#pragma unroll
        for (int j = 0; j < QPT; ++j) v[j] = top[p[j] + step - 1];
#pragma unroll
        for (int j = 0; j < QPT; ++j) p[j] = v[j] <= key[j] ? p[j] + step : p[j];
    }
    const uint32_t rlog2 = t.rlog2, nb = t.nb;
    bool found[QPT];
    uint32_t b[QPT];
#pragma unroll
    for (int j = 0; j < QPT; ++j) {
        const uint32_t cnt = p[j] < ntop ? p[j] : ntop;
        found[j] = cnt > 0 && x[j].x >= t.gmin;
        b[j] = (cnt > 0 ? cnt - 1 : 0) << rlog2;
    }
    if (rlog2 > 0) {
        // the 2^rlog2 buckets under the chosen LDS splitter (global, L2 resident)
        const K* gsplit = COMP ? reinterpret_cast<const K*>(t.split32)
                               : reinterpret_cast<const K*>(t.split64);
        const uint32_t R = 1u << rlog2;
#pragma unroll
        for (int j = 0; j < QPT; ++j) {
            uint32_t len = nb - b[j] < R ? nb - b[j] : R;
            uint32_t base = b[j];
            while (len > 1) {
                const uint32_t half = len >> 1;
                base = (gsplit[base + half] <= key[j]) ? base + half : base;
                len -= half;
            }
            b[j] = base;
        }
    }
    PairRec rec[QPT];
#pragma unroll
    for (int j = 0; j < QPT; ++j) rec[j] = load_rec(t.rec + b[j]);
#pragma unroll
    for (int j = 0; j < QPT; ++j) {
        uint8_t v = V_UNMAPPED;
        int32_t o = -1;
        const uint64_t L = x[j].y;
        if (found[j]) classify_in_bucket(rec[j], x[j].x, L < 1 ? 1 : L, v, o);
        if (DMA && v == V_ALLOW) {
            // the first range of a bucket starts at the bucket's splitter
            const bool second = rec[j].base1 <= x[j].x;
            const uint64_t st = second ? rec[j].base1 : t.split64[b[j]];
            const uint64_t en = second ? rec[j].end1 : rec[j].end0;
            if (x[j].x != st || L != en - st) v = V_INEXACT;
        }
        const uint64_t i = c0 + (uint64_t)j * 64u + lane;
        if (!TAIL || i < n) {
            verdict[i] = v;
            owner[i] = o;
        }
    }
}

// ---------------------------------------------------------------- packed 16-byte records
// Offsets inside a bucket (the second range's base, both ends) are below 2^32 whenever packed
// records are built, so after one 64-bit subtraction the classification runs on 32-bit values.
template <bool COMP, int LEVELS, int QPT, bool TAIL, bool DMA, bool LREC>
__device__ __forceinline__ void chunk_packed(const DevTable& t, const unsigned char* lds_raw,
                                             const uint32_t* ri, const ulonglong2 (&x)[QPT],
                                             uint64_t n, uint8_t* __restrict__ verdict,
                                             int32_t* __restrict__ owner, uint64_t c0,
                                             uint32_t lane) {
    using K = typename KeyT<COMP>::T;
    const uint32_t ntop = t.ntop;
    K key[QPT];
    uint32_t p[QPT];
    keys_and_starts<COMP, QPT>(t, ri, x, key, p);
    // unrolled lifting: every step is a constant, so the LDS reads use immediate offsets
    const K* top = reinterpret_cast<const K*>(lds_raw);
#pragma unroll
    for (int lv = LEVELS - 1; lv >= 0; --lv) {
        const uint32_t step = 1u << lv;
        K v[QPT];
#pragma unroll
        for (int j = 0; j < QPT; ++j) v[j] = (top + step - 1)[p[j]];
#pragma unroll
        for (int j = 0; j < QPT; ++j) p[j] += v[j] <= key[j] ? step : 0u;
    }
    uint32_t b[QPT];
    bool found[QPT];
    K sp[QPT];
#pragma unroll
    for (int j = 0; j < QPT; ++j) {
        const uint32_t cnt = p[j] < ntop ? p[j] : ntop;
        found[j] = cnt > 0 && x[j].x >= t.gmin;
        b[j] = cnt > 0 ? cnt - 1 : 0;
        sp[j] = top[b[j]];
    }
    uint4 r[QPT];
#pragma unroll
    for (int j = 0; j < QPT; ++j)
        r[j] = LREC ? reinterpret_cast<const uint4*>(lds_raw + t.lds_bytes)[b[j]] : t.nrec[b[j]];
    const uint32_t m1 = t.w1 >= 32 ? 0xFFFFFFFFu : (1u << t.w1) - 1u;
    const uint32_t sb = t.sb, w1 = t.w1;
    uint8_t* vp = verdict + c0 + lane;
    int32_t* op = owner + c0 + lane;
#pragma unroll
    for (int j = 0; j < QPT; ++j) {
        // offset from the bucket base; an address 2^32 or more past it is in no range of it
        const uint64_t rel64 = COMP ? (x[j].x - t.gmin) - ((uint64_t)sp[j] << t.shift)
                                    : x[j].x - (uint64_t)sp[j];
        const bool near = (uint32_t)(rel64 >> 32) == 0u;
        const uint32_t rel = (uint32_t)rel64;
        const uint32_t ob1 = (r[j].x & m1) << sb;
        const uint32_t oe0 = w1 >= 32 ? 0u : r[j].x >> w1;
        const bool second = rel >= ob1;
        const uint32_t oend = second ? r[j].y : oe0;
        const uint32_t meta = second ? r[j].w : r[j].z;
        const bool inside = found[j] && near && rel < oend;
        // inside a range, oend - rel >= 1, so max(len, 1) <= oend - rel iff len <= oend - rel
        const bool fits = (uint32_t)(x[j].y >> 32) == 0u && (uint32_t)x[j].y <= oend - rel;
        // DMA: the range starts at offset 0 (first) or ob1 (second) and must be taken whole
        const uint32_t ost = second ? ob1 : 0u;
        const bool exact = !DMA || (rel == ost && (uint32_t)x[j].y == oend - ost);
        const uint8_t v = !inside ? V_UNMAPPED
                                  : ((meta & 3u) != KIND_USER
                                         ? V_PROTECTED
                                         : (fits ? (exact ? V_ALLOW : V_INEXACT) : V_STRADDLE));
        const int32_t o = inside ? (int32_t)(meta >> 2) : -1;
        if (TAIL) {
            const uint64_t i = c0 + (uint64_t)j * 64u + lane;
            if (i < n) {
                verdict[i] = v;
                owner[i] = o;
            }
        } else {
            __builtin_nontemporal_store(v, vp + j * 64);  // written once, not read back
            __builtin_nontemporal_store(o, op + j * 64);
        }
    }
}

// Grid-stride loop over chunks of 64*QPT queries per wave, full chunks software-pipelined.
template <bool COMP, bool PACKED, int LEVELS, int QPT, bool DMA, bool LREC>
__global__ __launch_bounds__(VBLOCK) void k_validate(DevTable t, const ulonglong2* __restrict__ q,
                                                      uint64_t n, uint8_t* __restrict__ verdict,
                                                      int32_t* __restrict__ owner) {
    extern __shared__ __align__(16) unsigned char lds_raw[];
    if (t.nb == 0) {
        // empty table: everything is unmapped
        for (uint64_t i = (uint64_t)blockIdx.x * VBLOCK + threadIdx.x; i < n;
             i += (uint64_t)gridDim.x * VBLOCK) {
            verdict[i] = V_UNMAPPED;
            owner[i] = -1;
        }
        return;
    }
    const uint32_t lane = threadIdx.x & 63u;
    const uint64_t wave = ((uint64_t)blockIdx.x * VBLOCK + threadIdx.x) >> 6;
    const uint64_t nwaves = ((uint64_t)gridDim.x * VBLOCK) >> 6;
    constexpr uint64_t CHUNK = 64u * QPT;
    const uint64_t nfull = n / CHUNK * CHUNK;
    const uint64_t stride = nwaves * CHUNK;
    uint64_t c0 = wave * CHUNK;
    ulonglong2 x[QPT];
    const uint32_t* ri = reinterpret_cast<const uint32_t*>(lds_raw + t.radix_off);
    stage_index(reinterpret_cast<uint4*>(lds_raw), t.index, t.lds_bytes / 16 + (LREC ? t.nb : 0));
    if (c0 < nfull) load_chunk<QPT, false>(q, n, c0, lane, x);
    for (; c0 < nfull; c0 += stride) {
        ulonglong2 cur[QPT];
#pragma unroll
        for (int j = 0; j < QPT; ++j) cur[j] = x[j];
        if (c0 + stride < nfull) load_chunk<QPT, false>(q, n, c0 + stride, lane, x);
        if (PACKED)
            chunk_packed<COMP, LEVELS, QPT, false, DMA, LREC>(t, lds_raw, ri, cur, n, verdict, owner, c0,
                                                              lane);
        else
            chunk_wide<COMP, QPT, false, DMA>(t, lds_raw, ri, cur, n, verdict, owner, c0, lane);
    }
    if (c0 < n) {
        load_chunk<QPT, true>(q, n, c0, lane, x);
        if (PACKED)
            chunk_packed<COMP, LEVELS, QPT, true, DMA, LREC>(t, lds_raw, ri, x, n, verdict, owner, c0, lane);
        else
            chunk_wide<COMP, QPT, true, DMA>(t, lds_raw, ri, x, n, verdict, owner, c0, lane);
    }
}

template <bool COMP, bool PACKED, int LEVELS, int QPT, bool DMA, bool LREC>
static hipError_t launch_v(const DevTable& t, const DevInfo& d, const void* q, uint64_t n,
                           uint8_t* verdict, int32_t* owner, hipStream_t s) {
    const void* fn = reinterpret_cast<const void*>(&k_validate<COMP, PACKED, LEVELS, QPT, DMA, LREC>);
    const size_t lds = t.lds_bytes + (LREC ? (size_t)t.nb * 16 : 0);
    hipError_t e = hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize,
                                       (int)(lds > 0 ? lds : 16));
    if (e != hipSuccess) return e;
    int per_cu = 0;
    e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, fn, VBLOCK, lds);
    if (e != hipSuccess) return e;
    // with the records in LDS one workgroup a CU streams large batches faster than two (2^26 queries 242 /
    // 251 us, DMA 225 / 262), two the smaller ones (2^22: 14.2 / 15.4)
    if (per_cu < 1 || (LREC && n > (1ull << 24))) per_cu = 1;
    const uint64_t chunks = (n + 64u * QPT - 1) / (64u * QPT);
    const uint64_t want = (chunks + (VBLOCK / 64) - 1) / (VBLOCK / 64);
    uint64_t grid = (uint64_t)d.num_cu * per_cu;
    if (want < grid) grid = want;
    hipLaunchKernelGGL((k_validate<COMP, PACKED, LEVELS, QPT, DMA, LREC>), dim3((uint32_t)grid),
                       dim3(VBLOCK), lds, s, t, reinterpret_cast<const ulonglong2*>(q), n, verdict, owner);
    return hipGetLastError();
}

template <bool COMP, bool DMA, bool LREC, int QP>
static hipError_t launch_packed(const DevTable& t, const DevInfo& d, const void* q, uint64_t n,
                                uint8_t* verdict, int32_t* owner, hipStream_t s) {
    switch (t.lift) {
        case 2: return launch_v<COMP, true, 2, QP, DMA, LREC>(t, d, q, n, verdict, owner, s);
        case 4: return launch_v<COMP, true, 4, QP, DMA, LREC>(t, d, q, n, verdict, owner, s);
        case 6: return launch_v<COMP, true, 6, QP, DMA, LREC>(t, d, q, n, verdict, owner, s);
        default: return launch_v<COMP, true, 8, QP, DMA, LREC>(t, d, q, n, verdict, owner, s);
    }
}

// Records in LDS: a record read from L1 or L2 costs the CU's vector memory path one line per query (a
// line of 128 bytes at 64 bytes a clock, and a place among the lines it can have outstanding, which the
// query stream needs as well), a read from LDS neither. 2^26 queries, records in L2 / in LDS: 64 ranges 256 /
// 241 us, 4,096 354 / 242, 8,192 380 / 242, 12,000 395 / 243 (HBM alone 210). From 786,432 queries on, where
// staging them costs less than it saves (8,192 ranges, 700,001 queries 6.2 / 6.2, 1,000,003 6.7 / 6.1).
constexpr uint64_t LREC_MIN_N = 3ull << 18;
// Queries per lane: up to this many queries in a launch two, so that the chip's waves share them (200,000
// queries on 4,096 ranges 3.6 us, with six 6.1); beyond it eight, so that many record reads are in flight
// (2^26 on 65,536 ranges 424 us, with six 428, four 442, two 473). With the records in LDS two are best
// throughout (three 250, one 330 us against 242).
constexpr uint64_t FEW_N = 1ull << 20;

template <bool COMP, bool DMA>
static hipError_t launch_c(const DevTable& t, const DevInfo& d, const void* q, uint64_t n,
                           uint8_t* verdict, int32_t* owner, hipStream_t s) {
    if (t.narrow && t.rlog2 == 0) {  // then lift is 2, 4, 6 or 8
        if (t.lds_rec && n >= LREC_MIN_N)
            return launch_packed<COMP, DMA, true, 2>(t, d, q, n, verdict, owner, s);
        if (n <= FEW_N) return launch_packed<COMP, DMA, false, 2>(t, d, q, n, verdict, owner, s);
        return launch_packed<COMP, DMA, false, 8>(t, d, q, n, verdict, owner, s);
    }
    if (n <= FEW_N) return launch_v<COMP, false, 0, 2, DMA, false>(t, d, q, n, verdict, owner, s);
    return launch_v<COMP, false, 0, 6, DMA, false>(t, d, q, n, verdict, owner, s);
}

// ---------------------------------------------------------------- byte index (large tables)
// Tables whose records do not fit into LDS, where two bytes per range do (65,536 ranges: 150 KiB with the
// bins). The bin of an address and binary lifting over its ranges' low bytes give the range exactly, and
// its code two bounds of its size, between which most queries fall out the same. Only the lanes left open
// (a tenth of mixed pointer queries, 59% of DMA checks) read the range's end, so that the vector memory path is left to the
// streams. The vector units come next; hence 32-bit differences (ranges are shorter than 2^30 and start
// less than 2^31 apart) and no branch. 2^26 queries on 65,536 ranges 424 -> 264 us, DMA checks 429 -> 373
// (HBM alone 210; 302 / 282 / 276 with 2, 3 or 6 queries per lane, 327 with 64-bit differences and branches).
typedef __attribute__((address_space(3))) const uint8_t lds_u8;
typedef __attribute__((address_space(3))) const uint16_t lds_u16;

template <int QPT, bool DMA, bool TAIL>
__device__ __forceinline__ void chunk_bytes(const DevTable& t, const ByteIndex& x, uint32_t cbias,
                                            const ulonglong2 (&q)[QPT], uint64_t n,
                                            uint8_t* __restrict__ verdict, int32_t* __restrict__ owner,
                                            uint64_t c0, uint32_t lane) {
    // this kernel has no other LDS: offsets into the image are addresses
    lds_u8* low = (lds_u8*)0u;
    lds_u8* code = (lds_u8*)x.code_off;
    lds_u16* bin = (lds_u16*)x.bin_off;
    const uint32_t B = x.u + 8;
    uint32_t i[QPT], ql[QPT], i0[QPT], i1[QPT], before[QPT], dl[QPT];
    bool beyond[QPT], first_bin[QPT];
#pragma unroll
    for (int j = 0; j < QPT; ++j) {
        const uint64_t d = q[j].x - t.gmin;
        beyond[j] = d >= x.bins_end;
        dl[j] = (uint32_t)d;
        const uint32_t rd = __builtin_amdgcn_alignbit((uint32_t)(d >> 32), dl[j], B);
        const uint32_t r = rd < x.nbins - 1 ? rd : x.nbins - 1;
        ql[j] = __builtin_amdgcn_ubfe(dl[j], x.u, 8);
        first_bin[j] = r == 0;
        before[j] = bin[r];
        i[j] = i0[j] = bin[r + 1];
        i1[j] = bin[r + 2];
    }
    for (uint32_t step = (1u << x.levels) >> 1; step; step >>= 1) {
        uint32_t to[QPT], v[QPT];
#pragma unroll
        for (int j = 0; j < QPT; ++j) {
            to[j] = i[j] + step < i1[j] ? i[j] + step : i1[j];
            v[j] = low[to[j]];
        }
#pragma unroll
        for (int j = 0; j < QPT; ++j) i[j] = v[j] <= ql[j] ? to[j] : i[j];
    }
    uint32_t lo[QPT], c[QPT];
#pragma unroll
    for (int j = 0; j < QPT; ++j) {
        lo[j] = low[i[j]];
        c[j] = code[i[j]];
    }
    const __amdgpu_buffer_rsrc_t recs =
        __builtin_amdgcn_make_buffer_rsrc((void*)t.rec, 0, (int)(t.nb * sizeof(PairRec)), 0x00020000);
    bool first[QPT];
    uint32_t len[QPT], end[QPT], from[QPT];
#pragma unroll
    for (int j = 0; j < QPT; ++j) {
        // range i starts in an earlier bin: the one before, unless that has none (or is none: bin 0)
        const bool carry = (i[j] == i0[j]) & !(DMA & first_bin[j]);
        const bool known = !carry | (i[j] > before[j]);
        const uint32_t rel = (((carry ? 256u : 0u) - lo[j]) << x.u) + (dl[j] & ((1u << B) - 1));
        const uint32_t bits = ((c[j] & 127u) << x.csh) + cbias;
        const uint32_t sure = (uint32_t)__uint_as_float(bits);                 // <= size
        const uint32_t next = (uint32_t)__uint_as_float(bits + (1u << x.csh));  // > size
        // what is left of the range from the address on: at least rmin, less than rmax
        const int32_t rmin = (int32_t)(sure - rel), rmax = (int32_t)(next - rel);
        len[j] = (uint32_t)(q[j].y >> 32) ? ~0u : (uint32_t)q[j].y;
        first[j] = known & (rel == 0);
        const bool fits = (len[j] <= (uint32_t)rmin) & !(DMA & first[j] & (len[j] == sure));
        const bool in = (rmin > 0) & (fits | (len[j] > (uint32_t)rmax) | (c[j] > 127u));
        const bool open = !beyond[j] & !(known & (in | (rmax <= 0)));
        // a lane that is not open asks for an address past the buffer, which reads as zero, and goes on
        // with rmin (beyond the bins: with -1)
        const uint32_t at = (i[j] << 4) + ((~i[j] & 1u) << 3);
        end[j] = __builtin_amdgcn_raw_buffer_load_b32(recs, open ? at : 0x80000000u, 0, 0);
        const uint32_t closed = beyond[j] ? 1u : rel - sure;
        from[j] = open ? (uint32_t)q[j].x : closed;
    }
#pragma unroll
    for (int j = 0; j < QPT; ++j) {
        const int32_t room = (int32_t)(end[j] - from[j]);
        const bool whole = first[j] & (len[j] == (uint32_t)room);
        uint32_t v = DMA & !whole ? V_INEXACT : V_ALLOW;
        v = len[j] > (uint32_t)room ? V_STRADDLE : v;
        v = c[j] > 127u ? V_PROTECTED : v;
        v = room <= 0 ? V_UNMAPPED : v;
        const int32_t id = x.id0 + (int32_t)i[j], o = room <= 0 ? -1 : id;
        const uint64_t at = c0 + (uint64_t)j * 64u + lane;
        if (!TAIL || at < n) {
            __builtin_nontemporal_store((uint8_t)v, verdict + at);
            __builtin_nontemporal_store(o, owner + at);
        }
    }
}

template <int QPT, bool DMA>
__global__ __launch_bounds__(VBLOCK) void k_validate_bytes(DevTable t, ByteIndex x,
                                                            const ulonglong2* __restrict__ q, uint64_t n,
                                                            uint8_t* __restrict__ verdict,
                                                            int32_t* __restrict__ owner) {
    extern __shared__ __align__(16) unsigned char lds_raw[];
    stage_index(reinterpret_cast<uint4*>(lds_raw), x.image, x.bytes / 16);
    const uint32_t lane = threadIdx.x & 63u;
    uint32_t cbias;  // in a vector register: an instruction takes one scalar, here the shift
    asm("v_mov_b32 %0, %1" : "=v"(cbias) : "s"(x.cbias));
    constexpr uint64_t CHUNK = 64u * QPT;
    const uint64_t nfull = n / CHUNK * CHUNK, stride = (((uint64_t)gridDim.x * VBLOCK) >> 6) * CHUNK;
    uint64_t c0 = (((uint64_t)blockIdx.x * VBLOCK + threadIdx.x) >> 6) * CHUNK;
    ulonglong2 y[QPT], z[QPT];
    if (c0 < nfull) load_chunk<QPT, false>(q, n, c0, lane, y);
    while (c0 < nfull) {
        if (c0 + stride < nfull) load_chunk<QPT, false>(q, n, c0 + stride, lane, z);
        chunk_bytes<QPT, DMA, false>(t, x, cbias, y, n, verdict, owner, c0, lane);
        c0 += stride;
        if (c0 >= nfull) break;
        if (c0 + stride < nfull) load_chunk<QPT, false>(q, n, c0 + stride, lane, y);
        chunk_bytes<QPT, DMA, false>(t, x, cbias, z, n, verdict, owner, c0, lane);
        c0 += stride;
    }
    if (c0 < n) {
        load_chunk<QPT, true>(q, n, c0, lane, y);
        chunk_bytes<QPT, DMA, true>(t, x, cbias, y, n, verdict, owner, c0, lane);
    }
}

template <bool DMA>
static hipError_t launch_bytes(const DevTable& t, const ByteIndex& x, const DevInfo& d, const void* q,
                               uint64_t n, uint8_t* verdict, int32_t* owner, hipStream_t s) {
    constexpr int QPT = 4;
    const void* fn = reinterpret_cast<const void*>(&k_validate_bytes<QPT, DMA>);
    const hipError_t e = hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)x.bytes);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL((k_validate_bytes<QPT, DMA>), dim3((uint32_t)d.num_cu), dim3(VBLOCK), x.bytes, s, t, x,
                       reinterpret_cast<const ulonglong2*>(q), n, verdict, owner);
    return hipGetLastError();
}

hipError_t launch_validate(const DevTable& t, const ByteIndex& x, const DevInfo& d, const void* q,
                           uint64_t n, uint8_t* verdict, int32_t* owner, bool dma, hipStream_t s) {
    if (n == 0) return hipSuccess;
    if (x.bytes && n >= BYTES_MIN_N) {
        if (dma) return launch_bytes<true>(t, x, d, q, n, verdict, owner, s);
        return launch_bytes<false>(t, x, d, q, n, verdict, owner, s);
    }
    if (dma) {
        if (t.compressed) return launch_c<true, true>(t, d, q, n, verdict, owner, s);
        return launch_c<false, true>(t, d, q, n, verdict, owner, s);
    }
    if (t.compressed) return launch_c<true, false>(t, d, q, n, verdict, owner, s);
    return launch_c<false, false>(t, d, q, n, verdict, owner, s);
}

}  // namespace agile
