// Guarded streaming kernels: copy and the fp32 triad a = b + s*c (kernel memory guard of
// AgileOS Section V-E, with the suppress-and-record policies).
//
// Each pointer argument is bound once per call to the USER range containing it (a host lookup
// in the table the launch is ordered after), which turns the guard into an allowed prefix
// length per argument, passed in kernel arguments and so held in scalar registers. The vector
// loop compares each lane's vector offset with that bound before touching memory; vectors past
// a bound take the per-element path (denied loads read zero, denied stores are dropped). The
// denial count and the first denial follow in closed form from the prefix lengths: the caller works
// them out, with the first denial's reason, and one thread logs them. GUARD=false compiles the same loop with no compare (the unguarded twin).
#include "launch.h"

#pragma clang fp contract(off)

namespace agile {

constexpr int CBLOCK = 256, SBLOCK = 128;  // threads of the copy and the triad

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef u32x4 u32x4_any __attribute__((aligned(1)));  // a vector load at any address
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef f32x4 f32x4_any __attribute__((aligned(4)));

__device__ __forceinline__ void log_stream_fault(const StreamFault& f, DevLog* log,
                                                 unsigned long long seq) {
    if (f.count && blockIdx.x == 0 && threadIdx.x == 0) {
        atomicAdd(&log->count, (unsigned long long)f.count);
        log_record(log, seq, f.elem, f.operand, f.addr, f.width, f.op, f.verdict, f.owner);
    }
}

__device__ inline void copy_bytes_slow(uint8_t* dst, const uint8_t* src, uint64_t b0, uint64_t b1,
                                       uint64_t Ks, uint64_t Kd) {
    for (uint64_t k = b0; k < b1; ++k) {
        uint8_t v = k < Ks ? src[k] : (uint8_t)0;
        if (k < Kd) dst[k] = v;
    }
}

// Ks, Kd: allowed byte prefixes of src and dst (n and n for the unguarded twin). The first `up` bytes
// bring the destination to a 16-byte boundary; from there one vector per thread, stored aligned and
// loaded from wherever the source lies. 64 MiB: 22 us, from an odd address 24 us (126 with the one byte
// per thread that such a pointer took before), from one 4 bytes off 23 us (42 with 4-byte words).
template <bool GUARD>
__global__ __launch_bounds__(CBLOCK) void k_copy(StreamFault f, DevLog* log,
                                                  uint8_t* __restrict__ dst,
                                                  const uint8_t* __restrict__ src, uint64_t n,
                                                  uint64_t Ks, uint64_t Kd,
                                                  unsigned long long seq) {
    const uint64_t K = Ks < Kd ? Ks : Kd;
    const uint64_t tid = (uint64_t)blockIdx.x * CBLOCK + threadIdx.x;
    const uint64_t stride = (uint64_t)gridDim.x * CBLOCK;
    const uint64_t off = (0 - (uint64_t)dst) & 15, up = off < n ? off : n;
    const uint64_t nv = (n - up) / 16;
    const u32x4_any* sv = reinterpret_cast<const u32x4_any*>(src + up);
    u32x4* dv = reinterpret_cast<u32x4*>(dst + up);
    // vectors inside both allowed prefixes (they are prefixes, so one scalar bound covers them)
    const uint64_t in = K > up ? (K - up) / 16 : 0, lim = GUARD ? (in < nv ? in : nv) : nv;
    uint64_t v = tid;
    for (; v < lim; v += stride) __builtin_nontemporal_store(__builtin_nontemporal_load(sv + v), dv + v);
    // the guard's per-element path
    if (GUARD) {
        for (; v < nv; v += stride) {
            const uint64_t b0 = up + v * 16;
            if (b0 >= Ks && b0 + 16 <= Kd) dv[v] = u32x4{0u, 0u, 0u, 0u};
            else if (b0 < Kd) copy_bytes_slow(dst, src, b0, b0 + 16, Ks, Kd);
        }
    }
    // bytes before the first vector and after the last
    if (tid < up) copy_bytes_slow(dst, src, tid, tid + 1, Ks, Kd);
    const uint64_t tb = up + nv * 16 + tid;
    if (tb < n) copy_bytes_slow(dst, src, tb, tb + 1, Ks, Kd);
    if (GUARD) log_stream_fault(f, log, seq);
}

__device__ __forceinline__ float triad1(float b, float s, float c) {
    return __fadd_rn(b, __fmul_rn(s, c));
}

__device__ inline void triad_slow(float* a, const float* b, const float* c, float s, uint64_t i0,
                                  uint64_t i1, uint64_t Ka, uint64_t Kb, uint64_t Kc) {
    for (uint64_t i = i0; i < i1; ++i) {
        const float bv = i < Kb ? b[i] : 0.0f;
        const float cv = i < Kc ? c[i] : 0.0f;
        const float r = triad1(bv, s, cv);
        if (i < Ka) a[i] = r;
    }
}

// Ka, Kb, Kc: allowed element prefixes of the three operands (all n for the unguarded twin). The
// first `up` elements bring `a` to a 16-byte boundary; from there one vector per thread, b and c loaded
// from wherever they lie (2^25 elements: 61.5 us, one element off 67 us; with single elements 94 us).
template <bool GUARD>
__global__ __launch_bounds__(SBLOCK) void k_triad(StreamFault f, DevLog* log, float* a,
                                                   const float* b, const float* c, float s,
                                                   uint64_t n, uint64_t Ka, uint64_t Kb,
                                                   uint64_t Kc, unsigned long long seq) {
    uint64_t K = Ka < Kb ? Ka : Kb;
    K = K < Kc ? K : Kc;
    const uint64_t tid = (uint64_t)blockIdx.x * SBLOCK + threadIdx.x;
    const uint64_t stride = (uint64_t)gridDim.x * SBLOCK;
    const uint64_t off = ((0 - (uint64_t)a) & 15) / 4, up = off < n ? off : n;
    const uint64_t nv = (n - up) / 4;
    const f32x4_any* b4 = reinterpret_cast<const f32x4_any*>(b + up);
    const f32x4_any* c4 = reinterpret_cast<const f32x4_any*>(c + up);
    f32x4* a4 = reinterpret_cast<f32x4*>(a + up);
    const uint64_t in = K > up ? (K - up) / 4 : 0, lim = GUARD ? (in < nv ? in : nv) : nv;
    uint64_t v = tid;
    for (; v < lim; v += stride) {
        const f32x4 xb = __builtin_nontemporal_load(b4 + v);
        const f32x4 xc = __builtin_nontemporal_load(c4 + v);
        f32x4 r;
        r.x = triad1(xb.x, s, xc.x);
        r.y = triad1(xb.y, s, xc.y);
        r.z = triad1(xb.z, s, xc.z);
        r.w = triad1(xb.w, s, xc.w);
        __builtin_nontemporal_store(r, a4 + v);
    }
    if (GUARD) {
        for (; v < nv; v += stride) triad_slow(a, b, c, s, up + v * 4, up + v * 4 + 4, Ka, Kb, Kc);
    }
    if (tid < up) triad_slow(a, b, c, s, tid, tid + 1, Ka, Kb, Kc);
    const uint64_t ti = up + nv * 4 + tid;
    if (ti < n) triad_slow(a, b, c, s, ti, ti + 1, Ka, Kb, Kc);
    if (GUARD) log_stream_fault(f, log, seq);
}

// One pass: as many blocks as the vectors need, each thread one vector. Bound by HBM; measured on
// MI355X for 2^28 fp32 (triad) and 1 GiB (copy): 0.492 ms and 0.339 ms, against 0.540 ms and
// 0.382 ms with one persistent 256-thread workgroup per CU looping over 4 vectors per thread
// per pass (the hardware's block dispatch balances the end of the launch better than a fixed
// split), and against 0.51-0.60 ms for the triad with blocks of 64-256 threads and 2-4 vectors.
// One vector a thread, blocks of 128 / 256 threads: 256 MiB copy 83.9 / 83.7 us, from an odd address
// 90.2 / 89.6; triad of 2^25 61.5 / 62.8.
// As far as a grid holds it: from 2^32 vectors (64 GiB) on a thread takes further ones.
hipError_t launch_copy(bool guard, const StreamFault& f, DevLog* log, const Bind* binds, void* dst,
                       const void* src, uint64_t n, unsigned long long seq, hipStream_t s) {
    if (n == 0) return hipSuccess;
    const dim3 grid(workgroups(n / 16, CBLOCK, CBLOCK)), block(CBLOCK);
    if (guard)
        hipLaunchKernelGGL(k_copy<true>, grid, block, 0, s, f, log, (uint8_t*)dst, (const uint8_t*)src, n,
                           clip_prefix(binds[0], (uint64_t)src, n, 1),
                           clip_prefix(binds[1], (uint64_t)dst, n, 1), seq);
    else
        hipLaunchKernelGGL(k_copy<false>, grid, block, 0, s, f, log, (uint8_t*)dst, (const uint8_t*)src, n,
                           n, n, seq);
    return hipGetLastError();
}

hipError_t launch_triad(bool guard, const StreamFault& f, DevLog* log, const Bind* binds, float* a,
                        const float* b, const float* c, float sc, uint64_t n,
                        unsigned long long seq, hipStream_t s) {
    if (n == 0) return hipSuccess;
    const dim3 grid(workgroups(n / 4, SBLOCK, SBLOCK)), block(SBLOCK);
    if (guard)
        hipLaunchKernelGGL(k_triad<true>, grid, block, 0, s, f, log, a, b, c, sc, n,
                           clip_prefix(binds[2], (uint64_t)a, n, 4),
                           clip_prefix(binds[0], (uint64_t)b, n, 4),
                           clip_prefix(binds[1], (uint64_t)c, n, 4), seq);
    else
        hipLaunchKernelGGL(k_triad<false>, grid, block, 0, s, f, log, a, b, c, sc, n, n, n, n, seq);
    return hipGetLastError();
}

}  // namespace agile
