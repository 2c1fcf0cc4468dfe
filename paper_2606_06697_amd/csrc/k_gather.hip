// Guarded gather and scatter(-add) over rows (kernel memory guard of AgileOS Section V-E).
//
// out[i,:] = T[idx[i],:]  /  dst[idx[i],:] (+)= src[i,:], rows of `rb` bytes, elements of W bytes.
// The three pointer arguments are bound once per call (host lookup in the table the launch is
// ordered after) and reach the kernel as scalars. The index and the contiguous operand have
// prefix-shaped allowed sets; for the row-addressed operand the binding becomes an index
// interval [rlo, rhi] of rows that lie wholly inside the allocation, so the per-row guard is
// two signed compares of the loaded index against scalars. Rows outside it (hostile indices, or a table pointer that is not
// row-aligned with its allocation's ends) take an exact 128-bit per-element path. Denials are
// counted per lane, reduced per wave and folded into the handle's log (count and smallest
// (element, operand) key); the last workgroup, or a kernel after the launch, writes that denial's record.
// GUARD=false compiles the same loops with no binding and no compare (the unguarded twin).
#include "launch.h"

namespace agile {

constexpr int GBLOCK = 256;

template <int B>
struct Word;
template <>
struct Word<4> {
    using T = uint32_t;
};
template <>
struct Word<8> {
    using T = uint64_t;
};
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef u32x4 u32x4_any __attribute__((aligned(1)));  // a vector at any address
template <>
struct Word<16> {
    using T = u32x4_any;
};

// Lane layout shared by both kernels: a row is covered by G = 2^glog2 lanes (one CW-byte chunk
// each per pass), a wave covers 64/G rows, and each lane keeps R rows in flight. Rows of 16 bytes and
// more move in 16-byte chunks from any address; one that ends inside a chunk ends with a chunk that
// overlaps the one before, which is written with the same bytes (gathers of 1/4 GiB, against a chunk
// per element: 17 floats a row 325 -> 178 us, 33 297 -> 144, 65 217 -> 125, 255 160 -> 97, 5 390 -> 347;
// scatters of 2^19 rows of 17 floats 54 -> 35, 65 135 -> 86). WIDE kernels
// give a whole wave to each row (G = 64), so a row's index is wave-uniform and its guard test
// runs on scalar registers.
struct RowLanes {
    uint32_t G, lir, riw;
    uint64_t rpw, wave, nwaves;
    __device__ explicit RowLanes(uint32_t glog2) {
        const uint32_t lane = threadIdx.x & 63u;
        G = 1u << glog2;
        lir = lane & (G - 1);
        riw = lane >> glog2;
        rpw = 64u >> glog2;
        wave = ((uint64_t)blockIdx.x * GBLOCK + threadIdx.x) >> 6;
        nwaves = ((uint64_t)gridDim.x * GBLOCK) >> 6;
    }
};

// Per pass, every lane first issues the loads of all its rows that pass the fast test, then the
// matching stores, and only then runs the exact per-element path for the rest, so the guard
// adds no wait between the R independent loads. The fast test of row i is i < nfast (its index
// is readable and its contiguous-operand row is wholly allowed: both are prefixes) and
// rlo <= idx[i] <= rhi (its row-addressed row is wholly inside the binding). A row that has no byte in
// the binding needs no look at its elements either: a chunk of it is one store of zeros, or none, and
// one count (gathers of 131,072 rows of 256 floats with 1% / 30% / 100% denied 48 / 91 / 115 us element by
// element, now 38 / 38 / 38, and 36 without denials; scatters 48 / 90 / 108, now 38 / 37 / 29).
template <bool GUARD, bool WIDE, int R>
__device__ __forceinline__ void load_rows(const RowLanes& L, uint64_t r0, uint64_t nfast,
                                          const int64_t* idx, int64_t (&iv)[R]) {
#pragma unroll
    for (int u = 0; u < R; ++u) {
        const uint64_t i = r0 + u * L.rpw + L.riw;
        // narrow rows: each index is read once, non-temporally (kept out of L2 and the MALL,
        // which then hold more table lines); wide rows read one index per wave
        int64_t x = i < nfast ? (WIDE ? idx[i] : __builtin_nontemporal_load(idx + i)) : 0;
        if (WIDE) x = (int64_t)uniform_u64((uint64_t)x);
        iv[u] = x;
    }
}

template <bool GUARD, int CW, int W, int R, bool WIDE>
__global__ __launch_bounds__(GBLOCK) void k_gather(DevLog* log, uint8_t* out, const uint8_t* T,
                                                    uint64_t rb, const int64_t* idx, uint64_t n,
                                                    RowsGuard rg, int logon, uint32_t glog2,
                                                    FinishOf<GUARD> fin) {
    using V = typename Word<CW>::T;
    using E = typename Word<W>::T;
    constexpr uint32_t EPC = CW / W;  // elements per chunk
    const uint64_t D = rb / W;
    const uint64_t nch = (rb + CW - 1) / CW;
    const uint64_t Ki = rg.ki, Ko = rg.kc, nfast = rg.nfast;
    const RowGuard g = rg.g;
    const RowLanes L(WIDE ? 6u : glog2);
    FaultAcc acc;
    for (uint64_t r0 = L.wave * L.rpw * R; r0 < n; r0 += L.nwaves * L.rpw * R) {
        int64_t iv[R];
        load_rows<GUARD, WIDE, R>(L, r0, nfast, idx, iv);
        for (uint64_t c0 = 0; c0 < nch; c0 += L.G) {
            const uint64_t ch = c0 + L.lir;
            const uint64_t off = ch * CW < rb - CW ? ch * CW : rb - CW;
            V v[R];
            uint32_t slow = 0;  // rows of this lane whose chunk takes the exact path
#pragma unroll
            for (int u = 0; u < R; ++u) {
                const uint64_t i = r0 + u * L.rpw + L.riw;
                const bool on = i < n && ch < nch;
                const bool fast = on && (!GUARD || (i < nfast && g.rlo <= iv[u] && iv[u] <= g.rhi));
                if (fast) v[u] = *reinterpret_cast<const V*>(T + (uint64_t)iv[u] * rb + off);
                if (on && !fast) slow |= 1u << u;
            }
#pragma unroll
            for (int u = 0; u < R; ++u) {
                const uint64_t i = r0 + u * L.rpw + L.riw;
                if (i < n && ch < nch && !((slow >> u) & 1u))
                    __builtin_nontemporal_store(v[u], reinterpret_cast<V*>(out + i * rb + off));
            }
            if (!GUARD || slow == 0) continue;
#pragma unroll 1
            for (int u = 0; u < R; ++u) {
                if (!((slow >> u) & 1u)) continue;
                const uint64_t i = r0 + u * L.rpw + L.riw;
                const bool iok = i < Ki;
                if (!iok && ch == 0) acc.note((i * D) << 2);  // one 8-byte index load per row
                const int64_t x = iok ? idx[i] : 0;
                const uint64_t e0 = i * D + ch * EPC, ne = D - ch * EPC < EPC ? D - ch * EPC : EPC;
                if (row_outside(g, x) && e0 + ne <= Ko) {
                    *reinterpret_cast<V*>(out + i * rb + off) = V{};
                    acc.note_run((e0 << 2) | 1u, ne);
                    continue;
                }
                const bool full = g.rlo <= x && x <= g.rhi;
                const uint8_t* trow = T + (uint64_t)x * rb;
                uint8_t* orow = out + i * rb;
#pragma unroll 1
                for (uint64_t col = ch * EPC; col < D && col < (ch + 1) * EPC; ++col) {
                    const uint64_t e = i * D + col;
                    E val = 0;
                    if (full || elem_ok(g, x, rb, col, W)) {
                        val = *reinterpret_cast<const E*>(trow + col * W);
                    } else {
                        acc.note((e << 2) | 1u);
                    }
                    if (e < Ko) *reinterpret_cast<E*>(orow + col * W) = val;
                    else acc.note((e << 2) | 2u);
                }
            }
        }
    }
    if (GUARD && logon) end_faults(acc, log, fin);
}

// Plain scatter (no accumulation): with duplicate indices one of the writers wins.
template <bool GUARD, int CW, int W, int R, bool WIDE>
__global__ __launch_bounds__(GBLOCK) void k_scatter(DevLog* log, uint8_t* dst, uint64_t rb,
                                                     const int64_t* idx, const uint8_t* src,
                                                     uint64_t n, RowsGuard rg, int logon,
                                                     uint32_t glog2, FinishOf<GUARD> fin) {
    using V = typename Word<CW>::T;
    using E = typename Word<W>::T;
    constexpr uint32_t EPC = CW / W;
    const uint64_t D = rb / W;
    const uint64_t nch = (rb + CW - 1) / CW;
    const uint64_t Ki = rg.ki, Ks = rg.kc, nfast = rg.nfast;
    const RowGuard g = rg.g;
    const RowLanes L(WIDE ? 6u : glog2);
    FaultAcc acc;
    for (uint64_t r0 = L.wave * L.rpw * R; r0 < n; r0 += L.nwaves * L.rpw * R) {
        int64_t iv[R];
        load_rows<GUARD, WIDE, R>(L, r0, nfast, idx, iv);
        for (uint64_t c0 = 0; c0 < nch; c0 += L.G) {
            const uint64_t ch = c0 + L.lir;
            const uint64_t off = ch * CW < rb - CW ? ch * CW : rb - CW;
            V v[R];
            uint32_t slow = 0;
#pragma unroll
            for (int u = 0; u < R; ++u) {
                const uint64_t i = r0 + u * L.rpw + L.riw;
                const bool on = i < n && ch < nch;
                const bool fast = on && (!GUARD || (i < nfast && g.rlo <= iv[u] && iv[u] <= g.rhi));
                if (fast) v[u] = *reinterpret_cast<const V*>(src + i * rb + off);
                if (on && !fast) slow |= 1u << u;
            }
#pragma unroll
            for (int u = 0; u < R; ++u) {
                const uint64_t i = r0 + u * L.rpw + L.riw;
                if (i < n && ch < nch && !((slow >> u) & 1u))
                    *reinterpret_cast<V*>(dst + (uint64_t)iv[u] * rb + off) = v[u];
            }
            if (!GUARD || slow == 0) continue;
#pragma unroll 1
            for (int u = 0; u < R; ++u) {
                if (!((slow >> u) & 1u)) continue;
                const uint64_t i = r0 + u * L.rpw + L.riw;
                const bool iok = i < Ki;
                if (!iok && ch == 0) acc.note((i * D) << 2);
                const int64_t x = iok ? idx[i] : 0;
                const uint64_t e0 = i * D + ch * EPC, ne = D - ch * EPC < EPC ? D - ch * EPC : EPC;
                if (row_outside(g, x) && e0 + ne <= Ks) {
                    acc.note_run((e0 << 2) | 2u, ne);
                    continue;
                }
                const bool full = g.rlo <= x && x <= g.rhi;
                uint8_t* drow = dst + (uint64_t)x * rb;
                const uint8_t* srow = src + i * rb;
#pragma unroll 1
                for (uint64_t col = ch * EPC; col < D && col < (ch + 1) * EPC; ++col) {
                    const uint64_t e = i * D + col;
                    E val = 0;
                    if (e < Ks) val = *reinterpret_cast<const E*>(srow + col * W);
                    else acc.note((e << 2) | 1u);
                    if (full || elem_ok(g, x, rb, col, W)) {
                        *reinterpret_cast<E*>(drow + col * W) = val;
                    } else {
                        acc.note((e << 2) | 2u);
                    }
                }
            }
        }
    }
    if (GUARD && logon) end_faults(acc, log, fin);
}

// One wave: a place of the launches' denials per lane. The tickets are set up once, for a new log.
__global__ void k_log_reset(DevLog* log, uint32_t fresh) {
    if (fresh)
        for (uint32_t k = threadIdx.x; k < TICKET_WORDS / TICKET_STRIDE; k += FOLD_PLACES)
            log->ticket[k * TICKET_STRIDE] = 0;
    log->place[threadIdx.x].minkey = ~0ull;
    log->place[threadIdx.x].count = 0;
    if (threadIdx.x) return;
    log->count = 0;
    log->first_seq = ~0ull;
    log->first_elem = 0;
    log->first_addr = 0;
    log->first_width = 0;
    log->first_op = 0;
    log->first_operand = 0;
    log->first_verdict = 0;
    log->first_owner = -1;
    log->reserved = 0;
}

hipError_t launch_log_reset(DevLog* log, hipStream_t s, bool fresh) {
    hipLaunchKernelGGL(k_log_reset, dim3(1), dim3(FOLD_PLACES), 0, s, log, (uint32_t)fresh);
    return hipGetLastError();
}

// The finishing step as a kernel of its own (one wave), for launches that are not fused.
__global__ void k_fault_finish(DevTable t, DevLog* log, FaultSite f, unsigned long long seq) {
    finish_faults(ImageLook{t}, log, f, seq);
}
__global__ void k_fault_finish_inline(InlineTab t, DevLog* log, FaultSite f, unsigned long long seq) {
    finish_faults(InlineLook{t}, log, f, seq);
}

hipError_t launch_fault_finish(const GuardTab& t, DevLog* log, const FaultSite& f,
                               unsigned long long seq, hipStream_t s) {
    if (t.inl) hipLaunchKernelGGL(k_fault_finish_inline, dim3(1), dim3(64), 0, s, *t.inl, log, f, seq);
    else hipLaunchKernelGGL(k_fault_finish, dim3(1), dim3(64), 0, s, *t.dev, log, f, seq);
    return hipGetLastError();
}

// The workgroups count themselves up to this grid. With a finishing kernel / counted, gathers without denials
// and with 0.1%: 1,000 rows of 64 floats 8.7 / 5.8 us and 9.1 / 7.0, 2^19 rows of 4 bytes (1,024 workgroups)
// 9.5 / 7.4 and 11.4 / 10.2, 2^20 (2,048) 13.0 / 12.7 and 16.3 / 16.8, 2^22 (8,192) 76.2 / 75.5 and 80.8 / 80.8.
constexpr uint64_t FUSE_GRID = 2048;

FinishArgs finish_args(const GuardTab& t, const FaultSite& f, unsigned long long seq, uint64_t grid,
                       bool wanted, hipStream_t s) {
    static_assert(FUSE_GRID < 1u << TICKET_COUNT_BITS, "a word counts a launch's workgroups");
    FinishArgs a;
    a.fused = wanted && t.inl && grid <= FUSE_GRID && !is_captured(s);
    a.seq = seq;
    if (a.fused) {
        a.tab = *t.inl;
        a.site = f;
    }
    return a;
}

FaultSite rows_fault_site(uint32_t op, uint32_t w, uint32_t row_operand, uint64_t rb, uint64_t ki,
                          const void* idx, const void* cont, const void* rowp) {
    FaultSite f{};
    f.op = op;
    f.w = w;
    f.row_operand = row_operand;
    f.D = rb / w;
    f.rb = rb;
    f.ki = ki;
    f.idx = (uint64_t)idx;
    f.cont = (uint64_t)cont;
    f.rowp = (uint64_t)rowp;
    return f;
}

// Lanes per row: enough to cover the row's chunks, at most a wave.
static uint32_t lanes_log2(uint64_t nch) {
    uint32_t l = 0;
    while (l < 6 && (1ull << l) < nch) ++l;
    return l;
}

// Rows in flight per lane (R), by what a launch waits for. All on MI355X, us a call.
// - Few rows (the limits below): latency, so one or two rows and more workgroups; the kernel is also
//   shorter. 1,000 rows of 1 / 17 / 64 / 256 floats gathered 8.2 / 7.7 / 7.5 / 9.6 with R = 8 / 4 / 4 / 8,
//   now 6.8 / 6.9 / 6.5 / 7.3; 30,000 of 5 floats 8.5 -> 7.4, 100,000 of 256 38.8 -> 36.0.
// - Rows of at most 16 bytes, gathered: each load is a lone random access; from an allocation larger than
//   the L2s one pass of short-lived workgroups with one or two rows a lane beats eight (2^25 four-byte rows
//   of 2^28, 0.1% denied, 723 -> 682; 2^22 of 2^24 99 -> 91), from smaller ones eight are better beyond
//   2^20 rows (2^24 rows of 256 / 2^20: 173 / 194 against 202 / 217; of 2^22 284 / 297).
//   Scattered, beyond the limit: eight (2^20 rows of 8 / 12 / 16 bytes 29 / 35 / 32, with one or two
//   rows 33 / 40 / 37).
// - Rows below half a KiB: four (1/4 GiB of 17 / 33 / 64 floats 178 / 144 / 98; two rows 190 / 157 / 107).
// - Rows that take a whole wave, their index and guard in scalar registers: four (255 floats 97 -> 94, 129
//   doubles 124 -> 114 against eight). Two are best for uniform rows (92, 103), but 2^20 Zipf rows of 256
//   floats take 226 instead of 212, so only launches of up to 512 rows per CU take two (2^17 Zipf rows of
//   511 floats 89 -> 82).
//
// Grid: 4 workgroups per CU, the measured best of 1-16 for rows of a wave or more. Gathers of narrow rows
// go in one pass instead, with as many workgroups as the rows need: 1.437 ms against 1.458 ms for 2^26
// four-byte rows. The same change made the embedding's whole-wave rows slower (0.240 ms against 0.216 ms),
// so those keep the cap. One pass only as far as a grid holds it (2^31 twelve-byte or 2^33 four-byte rows of
// a large allocation): beyond that a wave takes further rows.
static uint32_t rows_grid(uint64_t n, uint32_t glog2, int R, const DevInfo& d,
                          bool one_pass = false) {
    const uint64_t rows_per_block = (uint64_t)(GBLOCK / 64) * (64u >> glog2) * R;
    return workgroups(n, rows_per_block, GBLOCK, one_pass ? ~0ull : (uint64_t)d.num_cu * 4);
}

struct RowCall {  // a row kernel's launch, and what its denials need
    GuardTab t;
    DevLog* log;
    uint64_t rb;
    const int64_t* idx;
    uint64_t n;
    RowsGuard rg;
    FaultSite site;
    unsigned long long seq;
    int logon;
    bool finish;
    DevInfo d;
    hipStream_t s;
};

// Launches the kernel, and the finishing kernel behind it where that is wanted and not fused.
template <bool G, class K, class L>
static hipError_t row_launch(const RowCall& c, K kernel, uint32_t grid, const L& launch) {
    const bool wanted = G && c.logon && c.finish;
    if constexpr (G) {
        const FinishArgs fin = finish_args(c.t, c.site, c.seq, grid, wanted, c.s);
        launch(kernel, grid, fin);
        if (wanted && !fin.fused) return launch_fault_finish(c.t, c.log, c.site, c.seq, c.s);
    } else {
        launch(kernel, grid, NoFinish{});
    }
    return hipGetLastError();
}

template <bool G, int CW, int W>
static hipError_t gather_cw(const RowCall& c, void* out, const void* tab) {
    const uint32_t gl = lanes_log2((c.rb + CW - 1) / CW);
    const auto launch = [&](auto k, uint32_t grid, const auto& fin) {
        hipLaunchKernelGGL(k, dim3(grid), dim3(GBLOCK), 0, c.s, c.log, (uint8_t*)out, (const uint8_t*)tab,
                           c.rb, c.idx, c.n, c.rg, c.logon, gl, fin);
    };
    if (gl == 6) {
        if (c.n <= (uint64_t)c.d.num_cu * 512)
            return row_launch<G>(c, k_gather<G, CW, W, 2, true>, rows_grid(c.n, gl, 2, c.d), launch);
        return row_launch<G>(c, k_gather<G, CW, W, 4, true>, rows_grid(c.n, gl, 4, c.d), launch);
    }
    if (c.rb <= 16) {
        constexpr int R = CW == 16 ? 1 : 2;
        const bool far = G && c.rg.g.bound && c.rg.g.rlo <= c.rg.g.rhi &&
                         (uint64_t)c.rg.g.rhi - (uint64_t)c.rg.g.rlo >= (32u << 20) / c.rb;
        if (far || c.n <= (uint64_t)c.d.num_cu * 4096)
            return row_launch<G>(c, k_gather<G, CW, W, R, false>, rows_grid(c.n, gl, R, c.d, true), launch);
        return row_launch<G>(c, k_gather<G, CW, W, 8, false>, rows_grid(c.n, gl, 8, c.d, true), launch);
    }
    if (c.n <= (uint64_t)c.d.num_cu * 16 * (64u >> gl))
        return row_launch<G>(c, k_gather<G, CW, W, 1, false>, rows_grid(c.n, gl, 1, c.d, true), launch);
    return row_launch<G>(c, k_gather<G, CW, W, 4, false>, rows_grid(c.n, gl, 4, c.d), launch);
}

template <bool G, int W>
static hipError_t gather_w(const RowCall& c, void* out, const void* tab) {
    if (c.rb >= 16) return gather_cw<G, 16, W>(c, out, tab);
    return gather_cw<G, W, W>(c, out, tab);
}

hipError_t launch_gather(bool guard, const GuardTab& t, DevLog* log, const Bind* binds, void* out,
                         const void* tab, uint64_t rb, const int64_t* idx, uint64_t n, uint32_t w,
                         unsigned long long seq, int logon, const DevInfo& d, hipStream_t s,
                         bool finish) {
    if (n == 0) return hipSuccess;
    RowCall c{t, log, rb, idx, n, rows_open(n, rb, w), FaultSite{}, seq, logon, finish, d, s};
    if (!guard) return w == 4 ? gather_w<false, 4>(c, out, tab) : gather_w<false, 8>(c, out, tab);
    c.rg = rows_guard(binds[0], binds[2], binds[1], (uint64_t)idx, (uint64_t)out, (uint64_t)tab, n, rb, w);
    c.site = rows_fault_site(3 /*OP_GATHER*/, w, 1, rb, c.rg.ki, idx, out, tab);
    return w == 4 ? gather_w<true, 4>(c, out, tab) : gather_w<true, 8>(c, out, tab);
}

template <bool G, int CW, int W>
static hipError_t scatter_cw(const RowCall& c, void* dst, const void* src) {
    const uint32_t gl = lanes_log2((c.rb + CW - 1) / CW);
    const auto launch = [&](auto k, uint32_t grid, const auto& fin) {
        hipLaunchKernelGGL(k, dim3(grid), dim3(GBLOCK), 0, c.s, c.log, (uint8_t*)dst, c.rb, c.idx,
                           (const uint8_t*)src, c.n, c.rg, c.logon, gl, fin);
    };
    if (gl == 6) {
        if (c.n <= (uint64_t)c.d.num_cu * 512)
            return row_launch<G>(c, k_scatter<G, CW, W, 2, true>, rows_grid(c.n, gl, 2, c.d), launch);
        return row_launch<G>(c, k_scatter<G, CW, W, 4, true>, rows_grid(c.n, gl, 4, c.d), launch);
    }
    if (c.rb <= 16) {
        constexpr int R = CW == 16 ? 1 : 2;
        if (c.n <= (uint64_t)c.d.num_cu * 1024)
            return row_launch<G>(c, k_scatter<G, CW, W, R, false>, rows_grid(c.n, gl, R, c.d), launch);
        return row_launch<G>(c, k_scatter<G, CW, W, 8, false>, rows_grid(c.n, gl, 8, c.d), launch);
    }
    if (c.n <= (uint64_t)c.d.num_cu * 16 * (64u >> gl))
        return row_launch<G>(c, k_scatter<G, CW, W, 1, false>, rows_grid(c.n, gl, 1, c.d, true), launch);
    return row_launch<G>(c, k_scatter<G, CW, W, 4, false>, rows_grid(c.n, gl, 4, c.d), launch);
}

template <bool G, int W>
static hipError_t scatter_w(const RowCall& c, void* dst, const void* src) {
    if (c.rb >= 16) return scatter_cw<G, 16, W>(c, dst, src);
    return scatter_cw<G, W, W>(c, dst, src);
}

hipError_t launch_scatter(bool guard, const GuardTab& t, DevLog* log, const Bind* binds, void* dst,
                          uint64_t rb, const int64_t* idx, const void* src, uint64_t n, uint32_t w,
                          int accumulate, unsigned long long seq, int logon, void* scratch,
                          const DevInfo& d, hipStream_t s, bool finish) {
    if (n == 0) return hipSuccess;
    if (accumulate)
        return launch_scatter_add(guard, t, log, binds, dst, rb, idx, src, n, w, seq, logon,
                                  scratch, d, s, finish, accumulate == 2);
    RowCall c{t, log, rb, idx, n, rows_open(n, rb, w), FaultSite{}, seq, logon, finish, d, s};
    if (!guard) return w == 4 ? scatter_w<false, 4>(c, dst, src) : scatter_w<false, 8>(c, dst, src);
    c.rg = rows_guard(binds[0], binds[1], binds[2], (uint64_t)idx, (uint64_t)src, (uint64_t)dst, n, rb, w);
    c.site = rows_fault_site(4 /*OP_SCATTER*/, w, 2, rb, c.rg.ki, idx, src, dst);
    return w == 4 ? scatter_w<true, 4>(c, dst, src) : scatter_w<true, 8>(c, dst, src);
}

}  // namespace agile
