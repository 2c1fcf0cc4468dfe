// Host-side launchers of the guard kernels (internal to libagile_guard.so).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "guard_device.h"
#include "launch_grid.h"

namespace agile {

struct DevInfo {
    int num_cu;
    size_t lds_per_block;  // largest dynamic LDS one workgroup may take
    size_t lds_per_cu;
};

// Maximum number of radix entries (plus one) the validation index may use.
constexpr uint32_t MAX_RADIX = (1u << 14) + 1;

// Least queries of a launch that uses the byte index, if the table has one. Smaller launches are over
// before the index (twice as long to stage) pays: 65,536 ranges, packed records in L2 against this, 2^19
// queries 6.2 / 7.1 us, 2^20 8.7 / 7.6, 2^21 15.6 / 10.9; DMA checks 6.3 / 7.3, 9.0 / 8.1, 15.6 / 12.4.
// Tables whose records fit the LDS are better off there: 8,192 ranges, 2^26 queries 242 against 269 us.
constexpr uint64_t BYTES_MIN_N = 1ull << 20;

// dma: answer the DMA registration check (only a whole USER range is ALLOW, else INEXACT).
hipError_t launch_validate(const DevTable& t, const ByteIndex& x, const DevInfo& d, const void* q,
                           uint64_t n, uint8_t* verdict, int32_t* owner, bool dma, hipStream_t s);

// The denials of a copy or triad, which follow from its allowed prefixes and are worked out by the
// caller (count == 0: none, or not logged); the launch writes them to the log.
struct StreamFault {
    uint64_t count, elem, addr;
    uint32_t width, op, operand, verdict;
    int32_t owner;
    uint32_t pad;
};

// The table that a row kernel's first denial is looked up in: in the launch's arguments, or (inl ==
// null) the uploaded image.
struct GuardTab {
    const DevTable* dev;
    const InlineTab* inl;
};

// Guarded launches take the bindings of their pointer arguments, looked up on the host from the
// table the launch is ordered after (`binds` in the operand order of the operation: copy src,
// dst; triad b, c, a; gather idx, table, out; scatter idx, src, dst). With guard == false
// `binds` is ignored and may be null.
hipError_t launch_copy(bool guard, const StreamFault& f, DevLog* log, const Bind* binds, void* dst,
                       const void* src, uint64_t n, unsigned long long seq, hipStream_t s);

hipError_t launch_triad(bool guard, const StreamFault& f, DevLog* log, const Bind* binds, float* a,
                        const float* b, const float* c, float sc, uint64_t n,
                        unsigned long long seq, hipStream_t s);

// finish == false leaves the launch's denials in the log scratch for a later kernel (the
// redirecting policies' pass) and the finishing kernel.
hipError_t launch_gather(bool guard, const GuardTab& t, DevLog* log, const Bind* binds, void* out,
                         const void* tab, uint64_t row_bytes, const int64_t* idx, uint64_t n,
                         uint32_t w, unsigned long long seq, int logon, const DevInfo& d,
                         hipStream_t s, bool finish = true);

// Scatter with accumulate = 1 uses `scratch` (device memory of at least
// scatter_add_scratch_bytes(n) bytes, or null for the chunk path) for its sort; calls that share
// a scratch buffer must be ordered on one stream.
hipError_t launch_scatter(bool guard, const GuardTab& t, DevLog* log, const Bind* binds, void* dst,
                          uint64_t row_bytes, const int64_t* idx, const void* src, uint64_t n,
                          uint32_t w, int accumulate, unsigned long long seq, int logon,
                          void* scratch, const DevInfo& d, hipStream_t s, bool finish = true);

// zero_dst: the destination rows are +0.0 before the call (scatter-add mode 2); the sorted path
// then writes each row's sum without reading the row.
hipError_t launch_scatter_add(bool guard, const GuardTab& t, DevLog* log, const Bind* binds,
                              void* dst, uint64_t rb, const int64_t* idx, const void* src,
                              uint64_t n, uint32_t w, unsigned long long seq, int logon,
                              void* scratch, const DevInfo& d, hipStream_t s, bool finish = true,
                              bool zero_dst = false);

size_t scatter_add_scratch_bytes(uint64_t n);

// Scatter-add calls that sort their destination keys (given scratch): of more than 2^18 rows, or of
// at least 2^15 rows and 96 MiB. Sorting costs ten launches, about 50 us, and then reads each row once
// and writes it once; the chunk path is one launch, but adds a row's sum once per chunk. Chunk against
// sorted, Zipf indices (all different): 32,768 x 64 floats 27 / 60 us (27 / 62), 65,536 x 256 57 / 74 (77 / 84),
// 131,072 x 64 41 / 67 (44 / 72), 131,072 x 256 90 / 90 (129 / 108), 262,144 x 64 64 / 76, 262,144 x 256 157 /
// 124. Beyond 2^18 rows (256 chunks) the hottest row's sum would be added up in more steps, and less exactly,
// than the sorted path does.
inline bool scatter_add_sorts(uint64_t n, uint64_t rb) {
    return n > (1u << 18) || (n >= (1u << 15) && n * rb > (96u << 20));
}

// fresh: a log that no launch has used yet.
hipError_t launch_log_reset(DevLog* log, hipStream_t s, bool fresh = false);

// Redirecting policies (sink to a quarantine, report): the pass after a guarded kernel.
constexpr uint32_t REDIRECT_SINK = 1, REDIRECT_REPORT = 2, REDIRECT_REMAP = 3;
struct Redirect {
    uint32_t mode;
    uint32_t pad;
    uint8_t* q;      // quarantine (SINK)
    uint64_t qmask;  // its size - 1 (a power of two)
};
// The bindings (REMAP rewrites into them) come in operand order.
struct RowBinds {
    Bind idx, cont, row;  // index array, contiguous operand (out / src), row-addressed operand
};
hipError_t launch_copy_fix(const DevTable& t, const Redirect& r, Bind bs, Bind bd, void* dst,
                           const void* src, uint64_t n, uint64_t Ks, uint64_t Kd, const DevInfo& d,
                           hipStream_t s);
hipError_t launch_triad_fix(const DevTable& t, const Redirect& r, Bind ba, Bind bb, Bind bc,
                            float* a, const float* b, const float* c, float sc, uint64_t n,
                            uint64_t Ka, uint64_t Kb, uint64_t Kc, const DevInfo& d,
                            hipStream_t s);
// op 0 gather (cont = out, rowp = table), 1 scatter, 2 scatter-add (cont = src, rowp = dst);
// rg: the guard over all n rows; the guarded kernel ran rows below rg.ki.
hipError_t launch_rows_fix(int op, const DevTable& t, DevLog* log, const Redirect& r,
                           const RowBinds& bb, void* cont, void* rowp, uint64_t rb,
                           const int64_t* idx, uint64_t n, const RowsGuard& rg, uint32_t w,
                           const DevInfo& d, hipStream_t s);

// After a guarded row kernel: folds the launch's denial count into the log and records the
// smallest key if the log is empty.
hipError_t launch_fault_finish(const GuardTab& t, DevLog* log, const FaultSite& f,
                               unsigned long long seq, hipStream_t s);
FaultSite rows_fault_site(uint32_t op, uint32_t w, uint32_t row_operand, uint64_t rb, uint64_t ki,
                          const void* idx, const void* cont, const void* rowp);
// Whether work queued on s becomes part of a graph (true also where that cannot be told).
inline bool is_captured(hipStream_t s) {
    hipStreamCaptureStatus c;
    if (hipStreamIsCapturing(s, &c) == hipSuccess) return c != hipStreamCaptureStatusNone;
    (void)hipGetLastError();
    return true;
}

// The finishing arguments of a launch of `grid` workgroups: fused when the table is in the arguments
// and the launch is small enough for its workgroups to count themselves. Launches that are captured end
// with the finishing kernel: replays of one launch share its number.
FinishArgs finish_args(const GuardTab& t, const FaultSite& f, unsigned long long seq, uint64_t grid,
                       bool wanted, hipStream_t s);

// ---- batched multi-client launch (device images of the public request/result layouts) ----
struct BatchReq {
    uint32_t client, reserved0;
    uint64_t ptr_off, nptr;
    uint64_t copy_dst, copy_src, copy_bytes;
    uint64_t gather_out, gather_table, gather_idx, gather_n;
    uint32_t gather_row_bytes, reserved1;
    uint64_t reserved2;
};
static_assert(sizeof(BatchReq) == 96, "BatchReq mirrors agile_request");

struct BatchScratch {
    unsigned int minfail;      // lowest failing pointer index of the request (or ~0)
    unsigned int remaining;    // pieces (workgroups) of the request not finished yet
    unsigned long long gcount; // gather denials
    unsigned long long gminkey;
    unsigned long long pad;
};
static_assert(sizeof(BatchScratch) == 32, "BatchScratch is 32 bytes");

struct agile_req_result_dev {
    uint32_t verdict;
    int32_t arg;
    int32_t owner;
    uint32_t done;
    unsigned long long fault_count, fault_seq, fault_elem, fault_addr;
    uint32_t fault_width, fault_op, fault_operand, fault_verdict;
    int32_t fault_owner;
    uint32_t fault_reserved;
};
static_assert(sizeof(agile_req_result_dev) == 72, "mirrors agile_req_result");

// Guard of one request, computed on the host from its client's table at launch time (the
// bindings of its copy and gather arguments as allowed prefixes and a row interval).
struct BatchGuard {
    uint64_t copy_ks, copy_kd;  // allowed byte prefixes of copy_src and copy_dst
    RowsGuard gather;           // gather: index / out prefixes and the table's row interval
};

struct BatchArgs {
    const uint64_t* tstart;  // nreq + 1 entries: first tile of each request, then the total
    const uint32_t* tile_req;  // ntiles entries: the request each tile belongs to
    const BatchGuard* guards;  // nreq entries
    const BatchReq* reqs;
    BatchScratch* scratch;
    const DevTable* tables;
    const ulonglong2* ptrs;
    uint8_t* pv;
    int32_t* po;
    agile_req_result_dev* result;
    uint64_t ntiles;
    uint64_t tile0;      // first tile of this launch
    uint64_t tile_copy;  // bytes per copy tile of this launch
    uint64_t tile_rows;  // rows per gather tile of this launch
    uint32_t nreq;
    uint32_t pad;
};

// Gather tiles of a request have 2^-batch_row_shift times the launch's rows per tile, so that a few thousand
// wide rows still spread over the chip. From 128 bytes on: with 64 / 128 / 256 here, a request of 50,000
// rows of 1 KiB takes 40 / 60 / 60 us a launch, one of 2,000 17 / 22 / 34, and 64 of 5,000 rows of 256 bytes 65
// / 37 / 44.
__host__ __device__ inline uint32_t batch_row_shift(const BatchReq& q) {
    uint32_t s = 0;
    while (s < 5 && q.gather_row_bytes > (128u << s)) ++s;
    return s;
}

// Tile sizes of one launch (rows counted 2^batch_row_shift times each), a request's tiles, and how many workgroups work on `tiles` of them.
void batch_tile_sizes(uint64_t copy_bytes, uint64_t gather_rows, uint64_t largest_gather,
                      uint64_t& tile_copy, uint64_t& tile_rows);
uint64_t batch_tiles(const BatchReq& q, uint64_t tile_copy, uint64_t tile_rows);
uint64_t batch_limit_tiles(const BatchReq& q);
uint32_t batch_pieces(uint64_t tiles);
hipError_t launch_batch(BatchArgs a, hipStream_t s);
hipError_t launch_batch_pull(void* dst, const void* src, uint64_t bytes, hipStream_t s);

}  // namespace agile
