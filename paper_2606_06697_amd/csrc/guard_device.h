// Device-side data layout and helpers shared by the guard kernels (gfx950, wave64).
//
// Table image (built on the host from the sorted range list, uploaded in stream order):
//   index       the validation's search index, laid out as it is staged in LDS (see DevTable)
//   nrec[b]     16 B the bucket's record with bit-packed offsets (see DevTable), when they fit
//   split64[b]  u64  base of the first range of bucket b (buckets hold 2 consecutive
//                    ranges in address order), nb = ceil(n/2) entries
//   split32[b]  u32  (split64[b] - gmin) >> shift, present when every bucket base is a
//                    multiple of 2^shift above gmin and the keys fit 32 bits; a query key
//                    (addr - gmin) >> shift then orders exactly like the address
//   rec[b]      32 B {base of the 2nd range (U64 max if none), end of 1st, end of 2nd,
//                    meta of 1st, meta of 2nd}, meta = id << 2 | kind
//   backed[b]   u8   bit 0 / bit 1: the first / second range was inserted as backed memory
// A lookup finds the last bucket whose base is <= addr, then reads one 32-byte record to
// pick the range inside the bucket and to get its end, id and kind.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

#include "guard_arith.h"
#include "ticket.h"

namespace agile {

constexpr uint32_t KIND_USER = 0;
constexpr uint8_t V_ALLOW = 0, V_PROTECTED = 1, V_STRADDLE = 2, V_UNMAPPED = 3,
                  V_CROSS_ALLOC = 4, V_INEXACT = 5;
constexpr uint64_t U64MAX = ~0ull;

struct alignas(32) PairRec {
    uint64_t base1;
    uint64_t end0;
    uint64_t end1;
    uint32_t meta0;
    uint32_t meta1;
};
static_assert(sizeof(PairRec) == 32, "PairRec is one 32-byte sector");

struct DevTable {
    const uint64_t* split64;
    const uint32_t* split32;
    const PairRec* rec;
    const uint4* index;     // validation search index, see below
    const uint8_t* backed;  // per bucket: bit 0 / bit 1 = first / second range is backed memory
    uint64_t gmin;
    uint32_t nb;          // number of buckets (0 for an empty table)
    uint32_t shift;
    uint32_t compressed;  // split32 valid
    // Validation search geometry. The LDS holds top[k] = splitter(k << rlog2), k < ntop, then
    // `pad` sentinels of the largest key value, then radix[r] = number of top entries below
    // gmin + (r << rsh), r <= nr (radix[nr] = ntop): an address with offset d = addr - gmin
    // has its answer among top[radix[r] ..], r = min(d >> rsh, nr - 1), at most 2^rlevels - 1
    // entries on. With compressed keys, r = min(key >> xs, nr - 1) (xs = rsh - shift, capped at
    // 31; nr == 1 whenever it would exceed 31). pad = 2^lift, lift >= rlevels.
    uint32_t ntop;
    uint32_t rlog2;
    uint32_t nr;
    uint32_t rsh;
    uint32_t xs;
    uint32_t rlevels;
    uint32_t lift;
    uint32_t pad;
    uint32_t lds_bytes;   // LDS one validation workgroup needs (top + sentinels + radix), the bytes
                          // at `index`; a multiple of 16
    uint32_t radix_off;   // where the radix entries start in it
    // Packed records (validation only, present when narrow != 0; then rlog2 == 0): per bucket
    // 16 bytes {u32 lo, u32 hi, u32 meta0, u32 meta1} with offsets relative to the bucket base:
    // lo = (second range's base >> sb) | (first range's end << w1), hi = second range's end. They lie
    // right behind the index.
    const uint4* nrec;
    uint32_t narrow;
    uint32_t sb;
    uint32_t w1;
    uint32_t lds_rec;     // the packed records fit the LDS behind the index
    uint32_t pad2;
};

// Byte index of a large table (validation of large batches, see chunk_bytes). Ranges are numbered in
// address order, with ids id0, id0 + 1, ...; their bases lie on multiples of 2^u above the first, and 256
// such units make a bin (up to the last range's end). In LDS:
//   low[i] (u8): range i's base inside its bin, in units
//   code[i] (u8): bit 7: not a USER range; bits 0-6: its size rounded down to the float whose bits are
//     (code << csh) + cbias
//   bin[r + 2] (u16): the last range of the bins up to r; bin[0] = bin[1] = 0
struct ByteIndex {
    const uint4* image;  // as it lies in LDS
    uint64_t bins_end;   // nbins << (u + 8)
    uint32_t bytes;      // of the image, a multiple of 16 (0: the table has none)
    uint32_t code_off, bin_off;
    uint32_t u, nbins;
    uint32_t levels;  // bits of the most ranges in a bin
    uint32_t csh, cbias;
    int32_t id0;
};

// Denials of some of a launch's waves.
constexpr uint32_t FOLD_PLACES = 64;
struct FaultPlace {
    unsigned long long minkey;  // min over (elem << 2 | operand)
    unsigned long long count;
    unsigned long long pad[30];
};

// Device copy of the public fault log (same field order as agile_fault) + per-launch scratch.
struct DevLog {
    unsigned long long count;
    unsigned long long first_seq;
    unsigned long long first_elem;
    unsigned long long first_addr;
    uint32_t first_width;
    uint32_t first_op;
    uint32_t first_operand;
    uint32_t first_verdict;
    int32_t first_owner;
    uint32_t reserved;
    uint32_t pad[50];
    // Scratch of one guarded launch, returned to its idle state by the launch's finishing step: its
    // denials, in FOLD_PLACES places a memory channel apart. A place takes about 12 ns an atomic, one
    // after another, and each wave with a denial adds to one: 2^24 four-byte rows of 2^26 gathered, 1% /
    // 30% / all of them denied, 1,208 / 1,632 / 1,590 us with a single place, 339 / 291 / 102 with 64.
    FaultPlace place[FOLD_PLACES];
    uint64_t ticket[TICKET_WORDS];  // workgroups that are done (last_workgroup)
};

// A table of at most INLINE_RANGES ranges in a launch's own arguments (entries in address order), for
// the reason of its first denial: as many as a wave has lanes, and 1.3 of the 4 KiB that arguments may take.
// After a change of the table a gather of 1,000 rows of 64 floats takes 7 us with 3 ranges, 16-22 with 103 and
// 26-31 with 4,003: those are uploaded, and a kernel of its own records the denials.
constexpr uint32_t INLINE_RANGES = 64;
struct InlineTab {
    uint32_t n;
    uint32_t pad;
    uint64_t base[INLINE_RANGES], end[INLINE_RANGES];
    uint32_t meta[INLINE_RANGES];  // id << 2 | kind
};

// Classification of `a` inside bucket b (split64[b] <= a is known): verdict + owner for a
// length-L query (L >= 1).
__device__ __forceinline__ void classify_in_bucket(const PairRec& r, uint64_t a, uint64_t L,
                                                   uint8_t& v, int32_t& owner) {
    const bool second = r.base1 <= a;
    const uint64_t end = second ? r.end1 : r.end0;
    const uint32_t meta = second ? r.meta1 : r.meta0;
    if (a >= end) {
        v = V_UNMAPPED;
        owner = -1;
        return;
    }
    owner = (int32_t)(meta >> 2);
    if ((meta & 3u) != KIND_USER) {
        v = V_PROTECTED;
    } else {
        v = (L <= end - a) ? V_ALLOW : V_STRADDLE;
    }
}

__device__ __forceinline__ PairRec load_rec(const PairRec* p) {
    const ulonglong2* q = reinterpret_cast<const ulonglong2*>(p);
    ulonglong2 x = q[0];
    ulonglong2 y = q[1];
    PairRec r;
    r.base1 = x.x;
    r.end0 = x.y;
    r.end1 = y.x;
    r.meta0 = (uint32_t)y.y;
    r.meta1 = (uint32_t)(y.y >> 32);
    return r;
}

// Last bucket with split64[b] <= a, or -1. One lane, binary search over global memory
// (used for single lookups in fault records).
__device__ inline int64_t bucket_search_lane(const DevTable& t, uint64_t a) {
    if (t.nb == 0 || t.split64[0] > a) return -1;
    uint32_t base = 0, len = t.nb;
    while (len > 1) {
        uint32_t half = len >> 1;
        base = (t.split64[base + half] <= a) ? base + half : base;
        len -= half;
    }
    return base;
}

__device__ inline void verdict_lane(const DevTable& t, uint64_t a, uint64_t len, uint8_t& v,
                                    int32_t& owner) {
    int64_t b = bucket_search_lane(t, a);
    if (b < 0) {
        v = V_UNMAPPED;
        owner = -1;
        return;
    }
    classify_in_bucket(load_rec(t.rec + b), a, len < 1 ? 1 : len, v, owner);
}

// Move a wave-uniform 64-bit value into scalar registers (readfirstlane works on 32-bit
// halves and returns int: widen through uint32_t so no sign bits leak into the high half).
__device__ __forceinline__ uint64_t uniform_u64(uint64_t x) {
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)x);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(x >> 32));
    return ((uint64_t)hi << 32) | lo;
}

// Reason recorded for a denied access at address a (already known to lie in [0, 2^64)).
__device__ inline void reason_lane(const DevTable& t, uint64_t a, uint32_t w, uint32_t& v,
                                   int32_t& owner) {
    uint8_t vv;
    verdict_lane(t, a, w, vv, owner);
    v = (vv == V_ALLOW) ? V_CROSS_ALLOC : vv;
}

// Write the first-fault record if the log has none yet (launches of one handle are ordered,
// so an earlier launch's record always wins).
__device__ inline void log_record(DevLog* log, unsigned long long seq, unsigned long long elem,
                                  uint32_t operand, uint64_t addr, uint32_t width, uint32_t op,
                                  uint32_t verdict, int32_t owner) {
    if (log->first_seq != ~0ull) return;
    log->first_elem = elem;
    log->first_addr = addr;
    log->first_width = width;
    log->first_op = op;
    log->first_operand = operand;
    log->first_verdict = verdict;
    log->first_owner = owner;
    __threadfence();
    log->first_seq = seq;
}

// Wave reductions (wave64).
__device__ __forceinline__ unsigned long long wave_sum_u64(unsigned long long x) {
    for (int o = 32; o > 0; o >>= 1) x += __shfl_xor(x, o, 64);
    return x;
}
__device__ __forceinline__ unsigned long long wave_min_u64(unsigned long long x) {
    for (int o = 32; o > 0; o >>= 1) {
        unsigned long long y = __shfl_xor(x, o, 64);
        x = y < x ? y : x;
    }
    return x;
}

// ---- denial accounting shared by the data-dependent guarded kernels ----
struct FaultAcc {
    unsigned long long cnt = 0;
    unsigned long long mk = ~0ull;
    __device__ __forceinline__ void note(unsigned long long key) {
        note_run(key, 1);
    }
    // n denials, the first of them with the smallest key
    __device__ __forceinline__ void note_run(unsigned long long key, uint64_t n) {
        cnt += n;
        mk = key < mk ? key : mk;
    }
};

// Fold per-lane denials into the launch's scratch: one atomic pair per wave that saw a denial
// (no workgroup-wide step, so waves and workgroups finish independently). The record of the
// smallest key is written afterwards by the launch's finishing step.
__device__ inline void fold_faults(FaultAcc acc, DevLog* log) {
    const unsigned long long c = wave_sum_u64(acc.cnt);
    const unsigned long long m = wave_min_u64(acc.mk);
    if ((threadIdx.x & 63u) == 0 && c) {
        FaultPlace* p = log->place + (blockIdx.x * 4u + (threadIdx.x >> 6)) % FOLD_PLACES;
        atomicAdd(&p->count, c);
        atomicMin(&p->minkey, m);
    }
}

// Where the denials of a row kernel (gather, scatter, scatter-add) live: a key's element e is
// row i = e / D, column e % D; operand 0 is the index load at idx + 8 i, the contiguous operand is
// at cont + e * w and the row-addressed one at rowp + idx[i] * rb + column * w.
struct FaultSite {
    uint32_t op;           // AGILE_OP_* of the call
    uint32_t w;            // element width
    uint32_t row_operand;  // operand number of the row-addressed pointer (1 gather, 2 scatter)
    uint32_t pad;
    uint64_t D, rb, ki;    // elements per row, row bytes, readable index prefix
    uint64_t idx, cont, rowp;
};

// What a launch of a row kernel needs to record its denials itself (fused != 0); otherwise a kernel
// after it does.
struct FinishArgs {
    InlineTab tab;
    FaultSite site;
    unsigned long long seq;
    uint32_t fused;
    uint32_t pad;
};
struct NoFinish {};  // the unguarded twins' place for it
template <bool GUARD>
using FinishOf = std::conditional_t<GUARD, FinishArgs, NoFinish>;

struct InlineLook {
    const InlineTab& t;
    // one range per lane of a wave
    __device__ __forceinline__ void operator()(uint64_t a, uint32_t w, uint32_t& v, int32_t& owner) const {
        static_assert(INLINE_RANGES == 64, "one range per lane");
        const uint32_t lane = threadIdx.x & 63u;
        const bool in = lane < t.n;
        const uint64_t base = in ? t.base[lane] : 0, end = in ? t.end[lane] : 0;
        const uint64_t m = __ballot(in && base <= a && a < end);
        v = V_UNMAPPED;
        owner = -1;
        if (!m) return;
        const uint32_t meta = __shfl(in ? t.meta[lane] : 0u, __builtin_ctzll(m), 64);
        const uint64_t room = __shfl(end, __builtin_ctzll(m), 64) - a;
        owner = (int32_t)(meta >> 2);
        v = (meta & 3u) != KIND_USER ? V_PROTECTED : (w <= room ? V_CROSS_ALLOC : V_STRADDLE);
    }
};
struct ImageLook {
    const DevTable& t;
    __device__ __forceinline__ void operator()(uint64_t a, uint32_t w, uint32_t& v, int32_t& owner) const {
        reason_lane(t, a, w, v, owner);
    }
};

// Finishing step of a row kernel's launch (one wave, a place of its denials per lane): adds the launch's
// denial count to the log and, if the log holds no record yet, records the smallest key (its address
// and reason).
template <class Look>
__device__ inline void finish_faults(const Look& look, DevLog* log, const FaultSite& f,
                                     unsigned long long seq) {
    static_assert(FOLD_PLACES == 64, "one place per lane");
    // the launch's waves folded into these from every XCD
    FaultPlace* mine = log->place + (threadIdx.x & 63u);
    const unsigned long long cnt =
        __hip_atomic_load(&mine->count, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    const unsigned long long low =
        __hip_atomic_load(&mine->minkey, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    const unsigned long long total = wave_sum_u64(cnt);
    if (total == 0) return;
    const unsigned long long key = wave_min_u64(low);
    const unsigned long long elem = key >> 2;
    const uint32_t operand = (uint32_t)(key & 3u);
    const uint64_t i = elem / f.D, col = elem % f.D;
    const int64_t* idx = reinterpret_cast<const int64_t*>(f.idx);
    __int128 A;
    uint32_t w = f.w;
    if (operand == 0) {
        A = (__int128)f.idx + (__int128)(8 * i);
        w = 8;
    } else if (operand == f.row_operand) {
        const int64_t v = i < f.ki ? idx[i] : 0;
        A = (__int128)f.rowp + (__int128)v * (__int128)f.rb + (__int128)(col * f.w);
    } else {
        A = (__int128)f.cont + (__int128)elem * f.w;
    }
    uint32_t v = V_UNMAPPED;
    int32_t o = -1;
    if (A >= 0 && A <= (__int128)U64MAX) look((uint64_t)A, w, v, o);
    if ((threadIdx.x & 63u) == 0) {
        atomicAdd(&log->count, total);
        log_record(log, seq, elem, operand, (uint64_t)A, w, f.op, v, o);
    }
    if (cnt) {
        atomicExch(&mine->count, 0ull);
        atomicExch(&mine->minkey, ~0ull);
    }
}

struct TicketAtomics {
    __device__ __forceinline__ void raise(uint64_t* w, uint64_t v) const {
        (void)__hip_atomic_fetch_max(w, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    __device__ __forceinline__ uint64_t add(uint64_t* w) const {
        return __hip_atomic_fetch_add(w, (uint64_t)1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
};

// End of a guarded row kernel, called by every thread of every workgroup of the launch: folds the
// denials, and in a fused launch the last workgroup to get here finishes them.
__device__ inline void end_faults(const FaultAcc& acc, DevLog* log, const FinishArgs& fin) {
    fold_faults(acc, log);
    if (!fin.fused) return;
    __shared__ uint32_t s_last;
    // every wave waits for its own atomics, then the workgroup is counted
    asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
    __syncthreads();
    if (threadIdx.x == 0)
        s_last = gridDim.x == 1 || last_workgroup(TicketAtomics{}, log->ticket, fin.seq, blockIdx.x, gridDim.x);
    __syncthreads();
    if (s_last && threadIdx.x < 64) finish_faults(InlineLook{fin.tab}, log, fin.site, fin.seq);
}
__device__ inline void end_faults(const FaultAcc&, DevLog*, const NoFinish&) {}

}  // namespace agile
