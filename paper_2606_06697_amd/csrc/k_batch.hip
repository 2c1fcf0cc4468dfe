// Batched multi-client requests in one launch.
//
// The paper's runtime assigns each client to a worker, and the worker checks every pointer
// argument of a mediated request against that client's own allocations before the real call
// (AgileOS Sections IV-B, IV-C, IV-F; a pointer valid for another client is not valid here,
// Section III). Here one launch serves many requests of many clients: every request is cut
// into tiles (pointer validation, guarded copy, guarded gather), a tile is worked on by SUB
// workgroups, and the workgroup that finishes a request's last piece writes the request's
// result: the lowest failing pointer argument and the request's fault record.
//
// Bound by the copies' memory traffic. One workgroup per piece, up to eight of them resident on a
// CU, so that the dependent descriptor loads of one (tile -> request -> data) overlap the copies of
// the others, and the hardware's dispatch balances the end of the launch. What a request writes goes
// out with agent-scope (write-through) stores, so a piece ends with a wait for its own stores and
// one relaxed counter update. 512 requests with 0.84 GB of copies, 300,000 pointers and 1.3 million
// gathered rows: 270 us a launch (a persistent workgroup per CU that claimed 2 MiB tiles and ended
// each with a device-scope fence, which writes back the XCD's L2: 565 us). Per piece of a copy, 32
// KiB in 8 vectors a thread 270 us, 16 KiB 289, 64 KiB 308, 8 KiB 360; 512 threads 285-305. Plain
// loads, since clients' sources are copied more than once: non-temporal ones 330 us; plain stores
// 326 us against non-temporal ones; without the agent scope the same 289.
#include <type_traits>

#include "launch.h"

namespace agile {

constexpr int BBLOCK = 256;
constexpr uint32_t SUB = 4;                     // workgroups per tile
constexpr uint64_t TILE_PTRS = 2048;            // pointers per validation tile
constexpr uint64_t TILE_COPY = 128ull << 10;    // bytes per copy tile (times a power of two)
constexpr uint64_t TILE_ROWS = 2048;            // rows per gather tile (times a power of two)
constexpr uint64_t MAP_TILES = 1ull << 16;      // launches of more tiles get larger ones
constexpr uint64_t SUB_PTRS = TILE_PTRS / SUB;
constexpr int VQ = SUB_PTRS / BBLOCK;           // pointer queries per lane
constexpr int COPY_U = 8;                       // 16-byte vectors in flight per thread
constexpr uint64_t COPY_PASS = (uint64_t)BBLOCK * COPY_U * 16;  // one pass of a workgroup
static_assert(SUB_PTRS == (uint64_t)VQ * BBLOCK && TILE_COPY == SUB * COPY_PASS, "one pass a piece");
constexpr uint32_t LDS_KEYS = 16384;            // bytes of bucket keys staged in LDS for the search

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef u32x4 u32x4_any __attribute__((aligned(1)));

__device__ inline void tiles_of(const BatchReq& q, uint64_t tile_copy, uint64_t& vt,
                                uint64_t& ct) {
    vt = (q.nptr + TILE_PTRS - 1) / TILE_PTRS;
    ct = (q.copy_bytes + tile_copy - 1) / tile_copy;
}

// Stores of a request's outputs: write-through to the agent's memory, so that once they are waited
// for, whoever reads the request's `done` finds them, with no cache write-back by the workgroup.
template <typename T>
__device__ __forceinline__ void store_out(T* p, T v) {
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// VQ pointer queries per lane, searched together (uniform trip count over the client table). Every
// 2^k-th bucket key is staged in LDS (k = 0 up to 4,096 buckets with 32-bit keys, 2,048 with 64-bit
// ones: 16 KiB, which leaves room for six workgroups a CU): one round of coalesced loads instead of
// a chain of dependent global loads per query. The last k levels are searched in global memory.
template <bool COMP>
__device__ inline void validate_tile(const DevTable& t, const ulonglong2* ptrs, uint64_t p0,
                                     uint64_t k0, uint64_t k1, uint8_t* pv, int32_t* po,
                                     uint32_t& minfail, void* lds) {
    using K = std::conditional_t<COMP, uint32_t, uint64_t>;
    constexpr uint32_t CAP = LDS_KEYS / sizeof(K);
    const uint32_t nb = t.nb;
    const K* gk = COMP ? reinterpret_cast<const K*>(t.split32) : reinterpret_cast<const K*>(t.split64);
    K* sk = static_cast<K*>(lds);
    uint32_t lg = 0;
    while (nb > (uint64_t)CAP << lg) ++lg;
    const uint32_t ns = nb ? ((nb - 1) >> lg) + 1 : 0;
#pragma unroll 4
    for (uint32_t k = threadIdx.x; k < ns; k += BBLOCK) sk[k] = gk[(uint64_t)k << lg];
    uint64_t a[VQ], L[VQ];
    K key[VQ];
    uint32_t base[VQ];
    bool live[VQ];
#pragma unroll
    for (int q = 0; q < VQ; ++q) {
        const uint64_t k = k0 + (uint64_t)q * BBLOCK + threadIdx.x;
        live[q] = k < k1;
        const ulonglong2 x = live[q] ? ptrs[p0 + k] : make_ulonglong2(0, 0);
        a[q] = x.x;
        L[q] = x.y < 1 ? 1 : x.y;
        base[q] = 0;
        // an address below the table is searched as key 0 and turned away afterwards
        const uint64_t d = x.x >= t.gmin ? x.x - t.gmin : 0;
        const uint64_t kk = COMP ? d >> t.shift : x.x;
        key[q] = COMP && kk > 0xFFFFFFFFull ? (K)0xFFFFFFFFu : (K)kk;
    }
    __syncthreads();
    for (uint32_t len = ns; len > 1;) {
        const uint32_t half = len >> 1;
#pragma unroll
        for (int q = 0; q < VQ; ++q) base[q] = sk[base[q] + half] <= key[q] ? base[q] + half : base[q];
        len -= half;
    }
#pragma unroll
    for (int q = 0; q < VQ; ++q) base[q] <<= lg;
    for (uint32_t step = (1u << lg) >> 1; step; step >>= 1) {
#pragma unroll
        for (int q = 0; q < VQ; ++q)
            if (base[q] + step < nb && gk[base[q] + step] <= key[q]) base[q] += step;
    }
#pragma unroll
    for (int q = 0; q < VQ; ++q) {
        if (!live[q]) continue;
        const uint64_t k = k0 + (uint64_t)q * BBLOCK + threadIdx.x;
        uint8_t v = V_UNMAPPED;
        int32_t o = -1;
        // the first bucket starts at gmin, and every address from there on is in one
        if (nb > 0 && a[q] >= t.gmin) classify_in_bucket(load_rec(t.rec + base[q]), a[q], L[q], v, o);
        store_out(pv + p0 + k, v);
        store_out(po + p0 + k, o);
        if (v != V_ALLOW && (uint32_t)k < minfail) minfail = (uint32_t)k;
    }
}

__device__ inline void copy_byte(uint8_t* dst, const uint8_t* src, uint64_t k, uint64_t Ks,
                                 uint64_t Kd) {
    const uint8_t x = k < Ks ? src[k] : (uint8_t)0;
    if (k < Kd) store_out(dst + k, x);
}

// Bytes [o0, o1) of a guarded copy whose arguments allow the prefixes Ks (src) and Kd (dst), at most
// COPY_PASS of them. The destination is brought to a 16-byte boundary by single bytes; then 16-byte
// vectors follow, loaded from wherever the source happens to lie.
__device__ inline void copy_tile(uint8_t* dst, const uint8_t* src, uint64_t o0, uint64_t o1,
                                 uint64_t Ks, uint64_t Kd) {
    const uint64_t K = Ks < Kd ? Ks : Kd;
    const uint64_t up = (16 - (((uint64_t)dst + o0) & 15)) & 15;
    const uint64_t h = o1 - o0 < up ? o1 : o0 + up;
    if (o0 + threadIdx.x < h) copy_byte(dst, src, o0 + threadIdx.x, Ks, Kd);
    const uint64_t e = o1 < K ? o1 : K;
    const uint32_t nv = e > h ? (uint32_t)((e - h) / 16) : 0;  // vectors inside both prefixes
    // global-address-space pointers: the request's addresses arrive as integers, and generic
    // pointers would give flat accesses
    typedef __attribute__((address_space(1))) const u32x4_any gcv;
    const gcv* sv = (const gcv*)(uintptr_t)(src + h);
    const __amdgpu_buffer_rsrc_t rd =
        __builtin_amdgcn_make_buffer_rsrc(dst + h, 0, (int)(nv * 16), 0x00020000);
    u32x4 x[COPY_U];
#pragma unroll
    for (int u = 0; u < COPY_U; ++u) {
        const uint32_t w = threadIdx.x + (uint32_t)u * BBLOCK;
        if (w < nv) x[u] = sv[w];
    }
#pragma unroll
    for (int u = 0; u < COPY_U; ++u) {
        const uint32_t w = threadIdx.x + (uint32_t)u * BBLOCK;
        // the resource ends after nv vectors; 2 | 16: non-temporal, agent scope
        if (w < nv) __builtin_amdgcn_raw_buffer_store_b128(x[u], rd, (int)(w * 16), 0, 2 | 16);
    }
    // past the first bound: zero vectors where only the source is denied, else byte by byte
    for (uint64_t b0 = h + 16 * ((uint64_t)nv + threadIdx.x); b0 < o1; b0 += 16 * BBLOCK) {
        const uint64_t b1 = b0 + 16 < o1 ? b0 + 16 : o1;
        if (b0 >= Ks && b0 + 16 <= b1 && b1 <= Kd) {
            store_out(reinterpret_cast<uint64_t*>(dst + b0), (uint64_t)0);
            store_out(reinterpret_cast<uint64_t*>(dst + b0) + 1, (uint64_t)0);
        } else if (b0 < Kd) {
            for (uint64_t k = b0; k < b1; ++k) copy_byte(dst, src, k, Ks, Kd);
        }
    }
}

// Columns c0, c0 + step, ... of row i of a guarded gather whose index is iv.
__device__ inline void gather_row(const BatchReq& q, const RowGuard& g, uint64_t D, uint64_t Ko,
                                  uint64_t i, int64_t iv, uint32_t c0, uint32_t step, FaultAcc& acc) {
    const uint64_t rb = q.gather_row_bytes;
    const bool full = g.rlo <= iv && iv <= g.rhi;
    const uint8_t* trow = reinterpret_cast<const uint8_t*>(q.gather_table) + (uint64_t)iv * rb;
    uint32_t* out = reinterpret_cast<uint32_t*>(q.gather_out);
    for (uint64_t col = c0; col < D; col += step) {
        const uint64_t e = i * D + col;
        uint32_t val = 0;
        if (full || elem_ok(g, iv, rb, col, 4)) val = *reinterpret_cast<const uint32_t*>(trow + col * 4);
        else acc.note((e << 2) | 1u);
        if (e < Ko) store_out(out + e, val);
        else acc.note((e << 2) | 2u);
    }
}

// Rows of at least 16 bytes: 2^gl lanes a row, each 16-byte vectors of it from any address; a row that ends
// inside a vector ends with one that overlaps the one before. Against one thread per row, a word at a time
// (launches, us): 50,000 rows of 64 / 256 / 1,024 words 107 / 369 / 2,104 -> 22 / 60 / 78, 64 requests of
// 5,000 rows of 16 / 128 words 105 / 855 -> 23 / 76, one of 2,000 rows of 256 words 343 -> 22. The lanes of a
// row also share its exact path: 50,000 rows of 64 / 256 words, all denied, 51 / 152 us (by one lane a row 510 /
// 7,945).
__device__ inline void gather_tile_wide(const BatchReq& q, const RowsGuard& rg, uint64_t i0, uint64_t i1,
                                        FaultAcc& acc) {
    constexpr int R = 4;  // rows in flight per lane
    const uint64_t rb = q.gather_row_bytes, D = rb / 4, nv = (D + 3) / 4;
    const int64_t* idx = reinterpret_cast<const int64_t*>(q.gather_idx);
    const uint8_t* T = reinterpret_cast<const uint8_t*>(q.gather_table);
    const __amdgpu_buffer_rsrc_t ro = __builtin_amdgcn_make_buffer_rsrc(
        reinterpret_cast<uint8_t*>(q.gather_out) + i0 * rb, 0, (int)((i1 - i0) * rb), 0x00020000);
    const RowGuard g = rg.g;
    uint32_t gl = 0;
    while (gl < 6 && (1ull << gl) < nv) ++gl;
    const uint32_t lir = threadIdx.x & ((1u << gl) - 1), rpp = BBLOCK >> gl;
    for (uint64_t r0 = i0 + (threadIdx.x >> gl); r0 < i1; r0 += (uint64_t)rpp * R) {
        int64_t iv[R];
        bool fast[R];
#pragma unroll
        for (int u = 0; u < R; ++u) {
            const uint64_t i = r0 + (uint64_t)u * rpp;
            iv[u] = i < i1 && i < rg.ki ? idx[i] : 0;
            fast[u] = i < i1 && i < rg.nfast;
        }
#pragma unroll
        for (int u = 0; u < R; ++u) fast[u] = fast[u] && g.rlo <= iv[u] && iv[u] <= g.rhi;
        for (uint64_t c = lir; c < nv; c += 1u << gl) {
            const uint64_t off = (c * 4 + 4 <= D ? c * 4 : D - 4) * 4;
            u32x4 v[R];
#pragma unroll
            for (int u = 0; u < R; ++u)
                if (fast[u]) v[u] = *reinterpret_cast<const u32x4_any*>(T + (uint64_t)iv[u] * rb + off);
#pragma unroll
            for (int u = 0; u < R; ++u)
                if (fast[u])
                    __builtin_amdgcn_raw_buffer_store_b128(
                        v[u], ro, (uint32_t)((r0 + (uint64_t)u * rpp - i0) * rb + off), 0, 2 | 16);
        }
#pragma unroll 1
        for (int u = 0; u < R; ++u) {
            const uint64_t i = r0 + (uint64_t)u * rpp;
            if (fast[u] || i >= i1) continue;
            if (lir == 0 && i >= rg.ki) acc.note((i * D) << 2);
            gather_row(q, g, D, rg.kc, i, iv[u], lir, 1u << gl, acc);
        }
    }
}

__device__ inline void gather_tile(const BatchReq& q, const RowsGuard& rg, uint64_t i0, uint64_t i1,
                                   FaultAcc& acc) {
    constexpr int R = 2;  // rows in flight per thread
    const uint64_t D = q.gather_row_bytes / 4;
    // the output of a tile within 31 bits
    if (D >= 4 && i1 - i0 <= 0x7FFFFFFFu / q.gather_row_bytes) return gather_tile_wide(q, rg, i0, i1, acc);
    const int64_t* idx = reinterpret_cast<const int64_t*>(q.gather_idx);
    const uint32_t* T = reinterpret_cast<const uint32_t*>(q.gather_table);
    uint32_t* out = reinterpret_cast<uint32_t*>(q.gather_out);
    const RowGuard g = rg.g;
    for (uint64_t r0 = i0 + threadIdx.x; r0 < i1; r0 += (uint64_t)BBLOCK * R) {
        int64_t iv[R];
        uint32_t v[R];
        bool fast[R];
#pragma unroll
        for (int u = 0; u < R; ++u) {
            const uint64_t i = r0 + (uint64_t)u * BBLOCK;
            iv[u] = i < i1 && i < rg.ki ? idx[i] : 0;
            fast[u] = D == 1 && i < i1 && i < rg.nfast;
        }
#pragma unroll
        for (int u = 0; u < R; ++u) {
            fast[u] = fast[u] && g.rlo <= iv[u] && iv[u] <= g.rhi;
            if (fast[u]) v[u] = T[iv[u]];
        }
#pragma unroll
        for (int u = 0; u < R; ++u) {
            const uint64_t i = r0 + (uint64_t)u * BBLOCK;
            if (fast[u]) {
                store_out(out + i, v[u]);
            } else if (i < i1) {
                if (i >= rg.ki) acc.note((i * D) << 2);
                gather_row(q, g, D, rg.kc, i, iv[u], 0, 1, acc);
            }
        }
    }
}

// Past this workgroup's caches: what other workgroups wrote through.
template <typename T>
__device__ __forceinline__ T load_out(const T* p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

__device__ __forceinline__ void wait_own_stores() {
    asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
}

// Result of request r, written by the workgroup that finished its last piece (one thread). A
// device-scope fence before `done` would write back and invalidate the XCD's whole L2 for each
// request (512 requests with no work at all took 39 us that way, 6 us this way), so the
// fields are written through as the outputs are, and waited for.
__device__ inline void finish_request(const BatchArgs& A, uint32_t r) {
    const BatchReq& q = A.reqs[r];
    const DevTable& t = A.tables[q.client];
    BatchScratch* s = A.scratch + r;
    agile_req_result_dev* res = A.result + r;
    const uint32_t mf = load_out(&s->minfail);
    const unsigned long long gc = load_out(&s->gcount), key = load_out(&s->gminkey);
    const bool fails = mf != 0xFFFFFFFFu;
    const uint32_t verdict = fails ? load_out(A.pv + q.ptr_off + mf) : V_ALLOW;
    const int32_t owner = fails ? load_out(A.po + q.ptr_off + mf) : -1;
    store_out(&res->verdict, verdict);
    store_out(&res->arg, fails ? (int32_t)mf : -1);
    store_out(&res->owner, owner);
    DevLog f{};
    f.first_seq = ~0ull;
    f.first_owner = -1;
    if (q.copy_bytes) {
        const uint64_t n = q.copy_bytes;
        const uint64_t Ks = A.guards[r].copy_ks, Kd = A.guards[r].copy_kd;
        const uint64_t cnt = (n - Ks) + (n - Kd);
        if (cnt) {
            f.count += cnt;
            const uint32_t operand = Ks <= Kd ? 0u : 1u;
            const uint64_t k = operand ? Kd : Ks;
            const uint64_t Aaddr = (operand ? q.copy_dst : q.copy_src) + k;
            uint32_t v;
            int32_t o;
            reason_lane(t, Aaddr, 1, v, o);
            f.first_seq = r;
            f.first_elem = k;
            f.first_addr = Aaddr;
            f.first_width = 1;
            f.first_op = 1;
            f.first_operand = operand;
            f.first_verdict = v;
            f.first_owner = o;
        }
    }
    if (gc) {
        f.count += gc;
        if (f.first_seq == ~0ull) {
            const uint64_t D = q.gather_row_bytes / 4;
            const unsigned long long elem = key >> 2;
            const uint32_t operand = (uint32_t)(key & 3u);
            const uint64_t i = elem / D, col = elem % D;
            __int128 Aa;
            uint32_t w = 4;
            if (operand == 0) {
                Aa = (__int128)q.gather_idx + (__int128)(8 * i);
                w = 8;
            } else if (operand == 1) {
                const uint64_t Ki = A.guards[r].gather.ki;
                const int64_t v = i < Ki ? reinterpret_cast<const int64_t*>(q.gather_idx)[i] : 0;
                Aa = (__int128)q.gather_table + (__int128)v * (__int128)q.gather_row_bytes +
                     (__int128)(col * 4);
            } else {
                Aa = (__int128)q.gather_out + (__int128)elem * 4;
            }
            uint32_t v = V_UNMAPPED;
            int32_t o = -1;
            if (Aa >= 0 && Aa <= (__int128)U64MAX) reason_lane(t, (uint64_t)Aa, w, v, o);
            f.first_seq = r;
            f.first_elem = elem;
            f.first_addr = (uint64_t)Aa;
            f.first_width = w;
            f.first_op = 3;
            f.first_operand = operand;
            f.first_verdict = v;
            f.first_owner = o;
        }
    }
    store_out(&res->fault_count, f.count);
    store_out(&res->fault_seq, f.first_seq);
    store_out(&res->fault_elem, f.first_elem);
    store_out(&res->fault_addr, f.first_addr);
    store_out(&res->fault_width, f.first_width);
    store_out(&res->fault_op, f.first_op);
    store_out(&res->fault_operand, f.first_operand);
    store_out(&res->fault_verdict, f.first_verdict);
    store_out(&res->fault_owner, f.first_owner);
    store_out(&res->fault_reserved, 0u);
    wait_own_stores();
    store_out(&res->done, 1u);
}

// Workgroup b works on piece b % SUB of tile b / SUB. Six waves a SIMD: one register more than their 80 and
// 512 mixed requests take 299 us instead of 287; bound to 64 they take 375.
__global__ __launch_bounds__(BBLOCK, 6) void k_batch(BatchArgs A) {
    __shared__ uint32_t s_minfail;
    __shared__ unsigned long long s_denied, s_mindenied;  // a gather piece's denials, least key
    __shared__ __align__(16) unsigned char s_keys[LDS_KEYS];
    const uint32_t tid = threadIdx.x;
    const uint64_t tile = A.tile0 + blockIdx.x / SUB;
    const uint32_t sub = blockIdx.x % SUB;
    const uint32_t r = A.tile_req[tile];
    const BatchReq& q = A.reqs[r];
    uint64_t vt, ct;
    tiles_of(q, A.tile_copy, vt, ct);
    const uint64_t local = tile - A.tstart[r];
    if (local < vt) {
        const uint64_t k0 = local * TILE_PTRS + sub * SUB_PTRS;
        const uint64_t k1 = k0 + SUB_PTRS < q.nptr ? k0 + SUB_PTRS : q.nptr;
        if (k0 < k1) {
            if (tid == 0) s_minfail = 0xFFFFFFFFu;
            __syncthreads();
            uint32_t mf = 0xFFFFFFFFu;
            const DevTable& t = A.tables[q.client];
            if (t.compressed) validate_tile<true>(t, A.ptrs, q.ptr_off, k0, k1, A.pv, A.po, mf, s_keys);
            else validate_tile<false>(t, A.ptrs, q.ptr_off, k0, k1, A.pv, A.po, mf, s_keys);
            if (mf != 0xFFFFFFFFu) atomicMin(&s_minfail, mf);
            __syncthreads();
            if (tid == 0 && s_minfail != 0xFFFFFFFFu) atomicMin(&A.scratch[r].minfail, s_minfail);
        }
    } else if (local < vt + ct) {
        // piece j of the copy takes passes j, j + SUB, ... of its tile
        const uint64_t t0 = (local - vt) * A.tile_copy;
        const uint64_t t1 = t0 + A.tile_copy < q.copy_bytes ? t0 + A.tile_copy : q.copy_bytes;
        for (uint64_t o0 = t0 + sub * COPY_PASS; o0 < t1; o0 += SUB * COPY_PASS)
            copy_tile(reinterpret_cast<uint8_t*>(q.copy_dst),
                      reinterpret_cast<const uint8_t*>(q.copy_src), o0,
                      o0 + COPY_PASS < t1 ? o0 + COPY_PASS : t1, A.guards[r].copy_ks,
                      A.guards[r].copy_kd);
    } else if (q.gather_n) {
        // the request's one count is touched once per workgroup: 2^20 rows of a word, 1% denied, 56 us (125
        // with two atomics per wave)
        if (tid == 0) {
            s_denied = 0;
            s_mindenied = ~0ull;
        }
        __syncthreads();
        const uint64_t tile_rows = A.tile_rows >> batch_row_shift(q), rows = tile_rows / SUB;
        const uint64_t i0 = (local - vt - ct) * tile_rows + sub * rows;
        const uint64_t i1 = i0 + rows < q.gather_n ? i0 + rows : q.gather_n;
        FaultAcc acc;
        gather_tile(q, A.guards[r].gather, i0, i1, acc);
        const unsigned long long c = wave_sum_u64(acc.cnt);
        const unsigned long long m = wave_min_u64(acc.mk);
        if ((tid & 63u) == 0 && c) {
            atomicAdd(&s_denied, c);
            atomicMin(&s_mindenied, m);
        }
        __syncthreads();
        if (tid == 0 && s_denied) {
            atomicAdd(&A.scratch[r].gcount, s_denied);
            atomicMin(&A.scratch[r].gminkey, s_mindenied);
        }
    }
    // every wave waits for its own write-through stores and atomics, then the piece is counted
    wait_own_stores();
    __syncthreads();
    if (tid == 0 && __hip_atomic_fetch_sub(&A.scratch[r].remaining, 1u, __ATOMIC_RELAXED,
                                           __HIP_MEMORY_SCOPE_AGENT) == 1u)
        finish_request(A, r);
}

hipError_t launch_batch(BatchArgs A, hipStream_t s) {
    constexpr uint64_t PART = 1ull << 20;  // tiles per launch: a grid has fewer than 2^32 threads
    for (uint64_t t = 0; t < A.ntiles; t += PART) {
        A.tile0 = t;
        const uint64_t n = A.ntiles - t < PART ? A.ntiles - t : PART;
        hipLaunchKernelGGL(k_batch, dim3((uint32_t)(n * SUB)), dim3(BBLOCK), 0, s, A);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

// Copies a launch's descriptors (about 150 KB for 512 requests) from the pinned staging buffer: a
// kernel in the launch's own queue starts and ends without the hand-over to and from a copy engine
// (289 us a launch against 323 with hipMemcpyAsync).
__global__ __launch_bounds__(BBLOCK) void k_batch_pull(u32x4* __restrict__ dst,
                                                       const u32x4* __restrict__ src, uint64_t n) {
    const uint64_t k = (uint64_t)blockIdx.x * BBLOCK + threadIdx.x;
    if (k < n) dst[k] = src[k];
}

hipError_t launch_batch_pull(void* dst, const void* src, uint64_t bytes, hipStream_t s) {
    const uint64_t n = (bytes + 15) / 16;  // the buffers are 64-byte padded
    hipLaunchKernelGGL(k_batch_pull, dim3((uint32_t)((n + BBLOCK - 1) / BBLOCK)), dim3(BBLOCK), 0, s,
                       static_cast<u32x4*>(dst), static_cast<const u32x4*>(src), n);
    return hipGetLastError();
}

// Tiles of one pass per workgroup, doubled until the launch's tile map has at most about MAP_TILES
// copy and as many gather tiles (4 GiB of copies, 2^27 rows): the map is written by the host and
// sent with each launch. Gather tiles are also doubled, up to 8,192 rows, while the largest gather has more
// than 64: a request's pieces count down one word, about 25 ns each one after another (a lone gather of
// 2^20 / 600,000 / 300,000 rows takes 44 / 35 / 28 us from launch to result, 55 / 42 / 30 in tiles of 2,048;
// one of 100,000 23, and 25 in tiles of 8,192. 512 requests with gathers of up to 65,536: 288, 295 with 8,192).
void batch_tile_sizes(uint64_t copy_bytes, uint64_t gather_rows, uint64_t largest_gather,
                      uint64_t& tile_copy, uint64_t& tile_rows) {
    tile_copy = TILE_COPY;
    while (tile_copy < (1ull << 40) && copy_bytes / tile_copy > MAP_TILES) tile_copy *= 2;
    tile_rows = TILE_ROWS;
    while (tile_rows < 4 * TILE_ROWS && largest_gather / tile_rows > 64) tile_rows *= 2;
    while (tile_rows < (1ull << 40) && gather_rows / tile_rows > MAP_TILES) tile_rows *= 2;
}

uint64_t batch_tiles(const BatchReq& q, uint64_t tile_copy, uint64_t tile_rows) {
    const uint64_t vt = (q.nptr + TILE_PTRS - 1) / TILE_PTRS;
    const uint64_t ct = (q.copy_bytes + tile_copy - 1) / tile_copy;
    const uint64_t rows = tile_rows >> batch_row_shift(q), gt = (q.gather_n + rows - 1) / rows;
    const uint64_t all = vt + ct + gt;
    return all ? all : 1;
}

// The tile count that bounds what one launch takes (2 MiB copy tiles, 16,384-row gather tiles).
uint64_t batch_limit_tiles(const BatchReq& q) {
    return (q.nptr + TILE_PTRS - 1) / TILE_PTRS + (q.copy_bytes + ((2ull << 20) - 1)) / (2ull << 20) +
           (q.gather_n + 16383) / 16384;
}

uint32_t batch_pieces(uint64_t tiles) { return (uint32_t)(tiles * SUB); }

}  // namespace agile
