// Client handle tokens: a worker-owned slot table behind opaque 64-bit tokens, so that forged,
// stale and cross-client handles are refused (AgileOS Section IV-C, the CUDA virtualization
// boundary), with a batched device check.
//
// Token = slot << 40 | gen << 16 | tag. The slot (24 bits) indexes the table; gen (24 bits) is
// the slot's generation when the token was minted; tag (16 bits) is the top of SplitMix64
// (Steele, Lea and Flood, 2014: state advanced by the golden gamma, then the published
// finalizer) of key ^ (slot << 24 | gen), under the table's secret key. Minting takes the
// lowest free slot; releasing advances the slot's generation, and a slot released in its last
// generation is retired.
//
// Device record per slot: {owner client, or FREE / RETIRED; gen << 8 | kind} in 8 bytes, or packed
// into 4 as long as the table's owners and generations leave room: kind in 8 bits, the owner in the
// next `ob` (its two largest values stand for FREE and RETIRED), the generation above. The
// host keeps the authoritative copy and uploads the dirty slot range in stream order before a
// check that follows a change; an owner or generation that outgrows its field changes the layout,
// and the whole table is uploaded again.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>
#include <new>
#include <set>
#include <vector>

#include "device_guard.h"
#include "agile_guard.h"

namespace agile {

constexpr uint32_t SLOT_MAX = 1u << 24;
constexpr uint32_t GEN_MASK = (1u << 24) - 1;
constexpr uint32_t OWNER_FREE = 0xFFFFFFFFu, OWNER_RETIRED = 0xFFFFFFFEu;
constexpr int TBLOCK = 256, LBLOCK = 1024;
constexpr int TPAIRS = 2;  // pairs of tokens per thread
// Least tokens of a launch that holds the slot records in LDS: 2^20 tokens take 7.4 us a call either way,
// 2^21 on 256 / 4,096 / 16,384 / 40,960 slots 8.0 / 8.2 / 8.1 / 8.9 with them there, 8.8 / 9.0 / 13.6 / 15.9 without.
constexpr uint64_t LREC_MIN_N = 1ull << 21;

static __host__ __device__ inline uint64_t splitmix64(uint64_t x) {
    uint64_t z = x + 0x9E3779B97F4A7C15ull;
    z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
    z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
    return z ^ (z >> 31);
}

static __host__ __device__ inline uint32_t token_tag(uint64_t key, uint32_t slot, uint32_t gen) {
    return (uint32_t)(splitmix64(key ^ (((uint64_t)slot << 24) | gen)) >> 48);
}

// One verdict; `rec` is the slot's record (read only when the slot is in range).
static __device__ __forceinline__ uint8_t token_verdict(uint64_t tok, uint32_t slot, uint2 rec, uint64_t key,
                                         uint32_t client, uint32_t want) {
    const uint32_t gen = (uint32_t)(tok >> 16) & GEN_MASK;
    if ((uint32_t)(tok & 0xFFFFu) != token_tag(key, slot, gen)) return AGILE_TOKEN_FORGED;
    const uint32_t rgen = rec.y >> 8, rkind = rec.y & 0xFFu;
    if (gen < rgen || rec.x == OWNER_RETIRED) return AGILE_TOKEN_STALE;
    if (gen > rgen || rec.x == OWNER_FREE) return AGILE_TOKEN_FORGED;
    if (rec.x != client) return AGILE_TOKEN_CROSS_CLIENT;
    if (want != AGILE_TOKEN_ANY_KIND && rkind != want) return AGILE_TOKEN_WRONG_KIND;
    return AGILE_TOKEN_VALID;
}

// How the slot records are laid out on the device: ob == 0 for 8 bytes, else packed.
struct RecLayout {
    uint32_t ob;
};

static __host__ __device__ inline uint32_t pack_rec(uint2 r, uint32_t ob) {
    // FREE and RETIRED, the two largest owners, are cut to the field's two largest values
    return (r.y >> 8) << (8 + ob) | (r.x & ((1u << ob) - 1)) << 8 | (r.y & 0xFFu);
}
static __host__ __device__ inline uint2 unpack_rec(uint32_t p, uint32_t ob) {
    const uint32_t free_code = (1u << ob) - 1, f = (p >> 8) & free_code;
    const uint32_t owner = f == free_code ? OWNER_FREE : f == free_code - 1 ? OWNER_RETIRED : f;
    return make_uint2(owner, (p >> (8 + ob)) << 8 | (p & 0xFFu));
}

typedef unsigned long long u64x2 __attribute__((ext_vector_type(2)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef u64x2 u64x2_at8 __attribute__((aligned(8)));
typedef u32x2 u32x2_at4 __attribute__((aligned(4)));
typedef uint16_t u16_any __attribute__((aligned(1)));

// One pass, TPAIRS pairs of neighbouring tokens per thread: a pair's tokens, clients and kinds are one
// load each and its verdicts and slots one store each (the vector memory path takes instructions in
// order, so fewer of them leave it to the record reads), and a thread's record reads, random ones of a
// table that the L2s hold, are issued together. The streams are non-temporal, so that they do not push
// the slot records out of L2. Bound by the vector memory path, on which record reads (a 128-byte line
// each, whatever the record's width) and streams do not overlap: 2^24 tokens over 2^20 slots take 130 us, the
// streams alone 48, the record reads alone 65, with the tokens' stream 88, with all streams in but none out
// 112, with those out but none in 58. 17 us are more than the two add up to; the size of the table is not
// the reason (2^18 slots, which fit L2 four times, 127). 141 with 8-byte records and four single tokens a
// thread; four pairs a thread 133.
//
// LREC: the packed records in LDS, staged by every workgroup, for large batches on tables that fit there
// (up to 40,960 slots). The record reads leave the vector memory path, and the streams bound it: 2^24
// tokens over 2^8 / 2^12 / 2^14 / 40,960 slots 50 / 50 / 51 / 52 us, from L1 and L2 64 / 64 / 99 / 118; with
// one or four pairs a thread 53-56 / 53-56 (and up to 16 / 17 instead of 13-15 for 2^22).
template <bool PACKED, bool LREC>
__global__ __launch_bounds__(LREC ? LBLOCK : TBLOCK) void k_tokens_check(
    const void* __restrict__ recs, uint32_t cap, RecLayout lay, uint64_t key,
    const uint64_t* __restrict__ tok, const uint32_t* __restrict__ cli,
    const uint8_t* __restrict__ kinds, uint64_t n, uint8_t* __restrict__ verdict,
    int32_t* __restrict__ slot_out) {
    extern __shared__ __align__(16) uint32_t lds_rec[];
    constexpr int TB = LREC ? LBLOCK : TBLOCK;
    if (LREC) {
#pragma unroll 1
        for (uint32_t k = threadIdx.x; k < (cap + 3) / 4; k += TB)
            reinterpret_cast<uint4*>(lds_rec)[k] = static_cast<const uint4*>(recs)[k];
        __syncthreads();
    }
    const auto record = [&](uint32_t s) {
        if (LREC) return unpack_rec(lds_rec[s], lay.ob);
        if (PACKED) return unpack_rec(static_cast<const uint32_t*>(recs)[s], lay.ob);
        return static_cast<const uint2*>(recs)[s];
    };
    const uint64_t np = n / 2, nth = (uint64_t)gridDim.x * TB;
    const uint64_t tid = (uint64_t)blockIdx.x * TB + threadIdx.x;
    for (uint64_t p0 = tid; p0 < np; p0 += nth * TPAIRS) {
        u64x2 t[TPAIRS];
        u32x2 c[TPAIRS];
        uint32_t w[TPAIRS];
        uint2 r[TPAIRS][2];
#pragma unroll
        for (int j = 0; j < TPAIRS; ++j) {
            // past the last pair: the last one again, not stored
            const uint64_t p = p0 + j * nth < np ? p0 + j * nth : np - 1;
            t[j] = __builtin_nontemporal_load(reinterpret_cast<const u64x2_at8*>(tok) + p);
            c[j] = __builtin_nontemporal_load(reinterpret_cast<const u32x2_at4*>(cli) + p);
            w[j] = kinds ? __builtin_nontemporal_load(reinterpret_cast<const u16_any*>(kinds) + p)
                         : AGILE_TOKEN_ANY_KIND * 0x101u;
        }
#pragma unroll
        for (int j = 0; j < TPAIRS; ++j)
#pragma unroll
            for (int q = 0; q < 2; ++q) {
                const uint32_t s = (uint32_t)(t[j][q] >> 40);
                r[j][q] = s < cap ? record(s) : make_uint2(OWNER_FREE, 0);
            }
#pragma unroll
        for (int j = 0; j < TPAIRS; ++j) {
            const uint64_t p = p0 + j * nth;
            uint32_t v[2];
            u32x2 so;
#pragma unroll
            for (int q = 0; q < 2; ++q) {
                const uint32_t s = (uint32_t)(t[j][q] >> 40);
                v[q] = s < cap ? token_verdict(t[j][q], s, r[j][q], key, c[j][q], (w[j] >> (8 * q)) & 0xFFu)
                               : (uint8_t)AGILE_TOKEN_FORGED;
                so[q] = v[q] == AGILE_TOKEN_VALID ? s : 0xFFFFFFFFu;
            }
            if (p < np) {
                __builtin_nontemporal_store((uint16_t)(v[0] | v[1] << 8),
                                            reinterpret_cast<u16_any*>(verdict) + p);
                __builtin_nontemporal_store(so, reinterpret_cast<u32x2_at4*>(slot_out) + p);
            }
        }
    }
    if ((n & 1) && tid == 0) {
        const uint64_t i = n - 1;
        const uint32_t s = (uint32_t)(tok[i] >> 40);
        const uint8_t v = s < cap ? token_verdict(tok[i], s, record(s), key, cli[i],
                                                  kinds ? kinds[i] : AGILE_TOKEN_ANY_KIND)
                                  : (uint8_t)AGILE_TOKEN_FORGED;
        verdict[i] = v;
        slot_out[i] = v == AGILE_TOKEN_VALID ? (int32_t)s : -1;
    }
}

}  // namespace agile

namespace {
using agile::DeviceGuard;
}  // namespace

using agile::GEN_MASK;
using agile::OWNER_FREE;
using agile::OWNER_RETIRED;
using agile::SLOT_MAX;
using agile::TBLOCK;
using agile::TPAIRS;
using agile::token_tag;

struct agile_tokens {
    int device = 0;
    uint32_t cap = 0;
    uint32_t num_cu = 0, lds = 0;     // compute units, most LDS of a workgroup
    uint64_t key = 0;
    std::vector<uint2> rec;           // authoritative slot records
    std::set<uint32_t> free_slots;    // released, reusable
    uint32_t next_new = 0;
    uint32_t dlo = 0, dhi = 0;        // dirty slot range [dlo, dhi)
    agile::RecLayout lay{10};         // packed until an owner or a generation asks for more
    uint32_t max_owner = 0, max_gen = 0;  // over every record written so far
    void* d_rec = nullptr;
    void* h_stage = nullptr;          // pinned staging of the upload
    hipEvent_t upload_done = nullptr;
    bool upload_pending = false;
    hipStream_t upload_stream = nullptr;
    bool uploaded = false;
    std::vector<hipStream_t> streams_used;  // streams that checked since the last upload
};

static void mark_dirty(agile_tokens* ts, uint32_t s) {
    if (ts->dlo >= ts->dhi) {
        ts->dlo = s;
        ts->dhi = s + 1;
    } else {
        ts->dlo = std::min(ts->dlo, s);
        ts->dhi = std::max(ts->dhi, s + 1);
    }
}

// Sets slot s's record; a value that its field cannot hold changes the layout of the device records.
static void set_rec(agile_tokens* ts, uint32_t s, uint2 r) {
    ts->rec[s] = r;
    mark_dirty(ts, s);
    if (r.x < OWNER_RETIRED) ts->max_owner = std::max(ts->max_owner, r.x);
    ts->max_gen = std::max(ts->max_gen, r.y >> 8);
    const auto fits = [&](uint32_t ob) {
        return (uint64_t)ts->max_owner + 2 < (1ull << ob) && (ts->max_gen >> (24 - ob)) == 0;
    };
    if (ts->lay.ob == 0 || fits(ts->lay.ob)) return;
    uint32_t ob = 2;  // the narrowest owner field, which leaves the generations the most room
    while (ob < 24 && (uint64_t)ts->max_owner + 2 >= (1ull << ob)) ++ob;
    ts->lay.ob = ob < 24 && fits(ob) ? ob : 0;
    ts->dlo = 0;
    ts->dhi = ts->cap;
}

int agile_tokens_create(agile_tokens** out, uint32_t capacity, uint64_t key, int device) {
    if (!out || capacity < 1 || capacity > SLOT_MAX) return AGILE_EINVAL;
    int ndev = 0;
    if (hipGetDeviceCount(&ndev) != hipSuccess) return AGILE_EDEVICE;
    if (device < 0 || device >= ndev) return AGILE_EINVAL;
    DeviceGuard dg(device);
    if (!dg.ok) return AGILE_EDEVICE;
    int num_cu = 0, lds = 0;
    if (hipDeviceGetAttribute(&num_cu, hipDeviceAttributeMultiprocessorCount, device) != hipSuccess ||
        hipDeviceGetAttribute(&lds, hipDeviceAttributeMaxSharedMemoryPerBlock, device) != hipSuccess)
        return AGILE_EDEVICE;
    agile_tokens* ts = new (std::nothrow) agile_tokens();
    if (!ts) return AGILE_ENOMEM;
    ts->num_cu = (uint32_t)num_cu;
    ts->lds = (uint32_t)lds;
    ts->device = device;
    ts->cap = capacity;
    ts->key = key;
    ts->rec.assign(capacity, make_uint2(OWNER_FREE, 0u));
    if (hipMalloc(&ts->d_rec, (size_t)capacity * sizeof(uint2)) != hipSuccess ||
        hipHostMalloc(&ts->h_stage, (size_t)capacity * sizeof(uint2),
                      hipHostMallocDefault) != hipSuccess ||
        hipEventCreateWithFlags(&ts->upload_done, hipEventDisableTiming) != hipSuccess) {
        agile_tokens_destroy(ts);
        return AGILE_ENOMEM;
    }
    ts->dlo = 0;
    ts->dhi = capacity;  // the first check uploads every (free) slot
    *out = ts;
    return AGILE_OK;
}

int agile_tokens_destroy(agile_tokens* ts) {
    if (!ts) return AGILE_OK;
    DeviceGuard dg(ts->device);
    int rc = AGILE_OK;
    if (hipDeviceSynchronize() != hipSuccess) rc = AGILE_EDEVICE;
    if (ts->upload_done) (void)hipEventDestroy(ts->upload_done);
    if (ts->h_stage) (void)hipHostFree(ts->h_stage);
    if (ts->d_rec) (void)hipFree(ts->d_rec);
    delete ts;
    return rc;
}

int agile_token_mint(agile_tokens* ts, uint32_t client, uint32_t kind, uint64_t* out_token) {
    if (!ts || !out_token || client >= OWNER_RETIRED || kind >= AGILE_TOKEN_ANY_KIND)
        return AGILE_EINVAL;
    uint32_t s;
    if (!ts->free_slots.empty()) {
        s = *ts->free_slots.begin();
        ts->free_slots.erase(ts->free_slots.begin());
    } else if (ts->next_new < ts->cap) {
        s = ts->next_new++;
    } else {
        return AGILE_ENOSPC;
    }
    const uint32_t gen = ts->rec[s].y >> 8;
    set_rec(ts, s, make_uint2(client, (gen << 8) | kind));
    *out_token = ((uint64_t)s << 40) | ((uint64_t)gen << 16) | token_tag(ts->key, s, gen);
    return AGILE_OK;
}

// Host-side verdict of one token (the same rule as the device check).
static int host_token_verdict(const agile_tokens* ts, uint64_t tok, uint32_t client, uint32_t* slot) {
    const uint32_t s = (uint32_t)(tok >> 40);
    if (s >= ts->cap) return AGILE_TOKEN_FORGED;
    *slot = s;
    const uint2 r = ts->rec[s];
    const uint32_t gen = (uint32_t)(tok >> 16) & GEN_MASK;
    if ((uint32_t)(tok & 0xFFFFu) != token_tag(ts->key, s, gen)) return AGILE_TOKEN_FORGED;
    if (gen < (r.y >> 8) || r.x == OWNER_RETIRED) return AGILE_TOKEN_STALE;
    if (gen > (r.y >> 8) || r.x == OWNER_FREE) return AGILE_TOKEN_FORGED;
    if (r.x != client) return AGILE_TOKEN_CROSS_CLIENT;
    return AGILE_TOKEN_VALID;
}

int agile_token_release(agile_tokens* ts, uint64_t token, uint32_t client) {
    if (!ts) return AGILE_EINVAL;
    uint32_t s = 0;
    if (host_token_verdict(ts, token, client, &s) != AGILE_TOKEN_VALID) return AGILE_ENOENT;
    const uint32_t gen = ts->rec[s].y >> 8;
    if (gen == GEN_MASK) {
        set_rec(ts, s, make_uint2(OWNER_RETIRED, gen << 8));
    } else {
        set_rec(ts, s, make_uint2(OWNER_FREE, (gen + 1) << 8));
        ts->free_slots.insert(s);
    }
    return AGILE_OK;
}

// Bring the device records up to date on stream s (in stream order).
static int tokens_prepare(agile_tokens* ts, hipStream_t s) {
    if (ts->dlo < ts->dhi) {
        // checks queued on other streams read the records about to be overwritten
        for (hipStream_t o : ts->streams_used) {
            if (o == s) continue;
            hipEvent_t ev;
            if (hipEventCreateWithFlags(&ev, hipEventDisableTiming) != hipSuccess) return AGILE_EDEVICE;
            const bool ok = hipEventRecord(ev, o) == hipSuccess && hipStreamWaitEvent(s, ev, 0) == hipSuccess;
            (void)hipEventDestroy(ev);
            if (!ok) return AGILE_EDEVICE;
        }
        ts->streams_used.clear();
        // the staging buffer may still feed the previous upload
        if (ts->upload_pending && hipEventSynchronize(ts->upload_done) != hipSuccess)
            return AGILE_EDEVICE;
        const size_t lo = ts->dlo, cnt = (size_t)ts->dhi - ts->dlo;
        const size_t w = ts->lay.ob ? sizeof(uint32_t) : sizeof(uint2);
        if (ts->lay.ob) {
            uint32_t* __restrict__ st = static_cast<uint32_t*>(ts->h_stage) + lo;
            const uint2* __restrict__ r = ts->rec.data() + lo;
            const uint32_t ob = ts->lay.ob;
            for (size_t k = 0; k < cnt; ++k) st[k] = agile::pack_rec(r[k], ob);
        } else {
            std::copy(ts->rec.begin() + lo, ts->rec.begin() + lo + cnt,
                      static_cast<uint2*>(ts->h_stage) + lo);
        }
        if (hipMemcpyAsync(static_cast<uint8_t*>(ts->d_rec) + lo * w,
                           static_cast<const uint8_t*>(ts->h_stage) + lo * w, cnt * w,
                           hipMemcpyHostToDevice, s) != hipSuccess ||
            hipEventRecord(ts->upload_done, s) != hipSuccess)
            return AGILE_EDEVICE;
        ts->upload_pending = true;
        ts->upload_stream = s;
        ts->uploaded = true;
        ts->dlo = ts->dhi = 0;
    } else if (ts->uploaded && ts->upload_stream != s) {
        if (hipStreamWaitEvent(s, ts->upload_done, 0) != hipSuccess) return AGILE_EDEVICE;
    }
    if (std::find(ts->streams_used.begin(), ts->streams_used.end(), s) == ts->streams_used.end())
        ts->streams_used.push_back(s);
    return AGILE_OK;
}

int agile_tokens_check(agile_tokens* ts, const uint64_t* d_tokens, const uint32_t* d_clients,
                       const uint8_t* d_kinds, uint64_t n, uint8_t* d_verdict, int32_t* d_slot,
                       void* stream) {
    if (!ts) return AGILE_EINVAL;
    if (n == 0) return AGILE_OK;
    if (!d_tokens || !d_clients || !d_verdict || !d_slot || ((uint64_t)d_tokens & 7) ||
        ((uint64_t)d_clients & 3) || ((uint64_t)d_slot & 3))
        return AGILE_EINVAL;
    DeviceGuard dg(ts->device);
    if (!dg.ok) return AGILE_EDEVICE;
    hipStream_t s = static_cast<hipStream_t>(stream);
    const int rc = tokens_prepare(ts, s);
    if (rc != AGILE_OK) return rc;
    const bool lrec = ts->lay.ob && ts->cap >= 4 && ts->cap <= ts->lds / 4 && n >= agile::LREC_MIN_N;
    const uint64_t tb = lrec ? agile::LBLOCK : TBLOCK, per_block = tb * TPAIRS;
    const size_t lds = lrec ? ((size_t)ts->cap + 3) / 4 * 16 : 0;
    uint64_t grid = (n / 2 + per_block - 1) / per_block;
    // one pass (2^26 tokens took 4% longer with 8 workgroups per CU looping); with the records in LDS one
    // workgroup per CU (2^24 tokens on 256 / 16,384 slots 50 / 50 us, with two 54 / 56)
    const uint64_t cap = lrec ? ts->num_cu : 1ull << 23;
    if (grid > cap) grid = cap;
    if (grid < 1) grid = 1;
    auto k = lrec ? agile::k_tokens_check<true, true>
                  : ts->lay.ob ? agile::k_tokens_check<true, false> : agile::k_tokens_check<false, false>;
    if (lrec && hipFuncSetAttribute(reinterpret_cast<const void*>(k),
                                    hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds) != hipSuccess)
        return AGILE_EDEVICE;
    hipLaunchKernelGGL(k, dim3((uint32_t)grid), dim3((uint32_t)tb), lds, s, ts->d_rec, ts->cap, ts->lay,
                       ts->key, d_tokens, d_clients, d_kinds, n, d_verdict, d_slot);
    return hipGetLastError() == hipSuccess ? AGILE_OK : AGILE_EDEVICE;
}
