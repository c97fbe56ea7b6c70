// qap_lap_solve: the batched assignment solve with canonical dual that every
// cost concentration performs (Section 4.1 of arXiv 1510.02065), offered on
// its own for host or device buffers.
//
// A batch that the chip holds at once runs as one launch, a wave per problem.
// Larger ones run in size classes, one launch each with segments of 16, 32 or
// 64 lanes per problem (4, 2 or 1 problems per wave), so that small problems
// do not each occupy a whole wave.  Within a class the problems go by falling size: a wave's
// problems then mostly have one size (its loop counts are scalars and none of
// its problems waits for a larger one), and the launch ends on short ones.
// With host buffers the host sorts the problems; with device buffers (whose
// sizes the host does not read) a device pass writes the order into a workspace
// and each class's launch reads its range from there.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <mutex>
#include <string>
#include <vector>

#include "handle.hpp"

using qap::fail;

namespace qap {

// Size classes of a batch, one launch each.  A launch's width (lanes per
// problem) and LDS are those of its largest size, and the next one starts when
// its last problem is done, so classes cost latency and save lanes and LDS.
// Measured (us, problems of uniform sizes, FP64 | FP32):
//   classes up to      64           16,32,64     16,32,48,64  16,32,48,56,64
//   1000 of 2..64      125 | 115    186 | 163
//   1000 of 3..14       46 |  53     52 |  56
//   4000 of 2..64      185 | 128    239 | 182
//   6000 of 3..14       95 |  71     80 |  74     73 |  83     85 |  83
//   6000 of 2..64      258 | 142    304 | 203    336 | 256    391 | 325
//   20000 of 2..64     807 | 347    752 | 366    716 | 392    731 | 432
//   20000 of 2..30     355 | 178    172 | 136    178 | 146    186 | 150
//   20000 of 33..50   1024 | 449   1039 | 458    748 | 401    721 | 403
//   40000 of 50..64   3026 | 1254  3040 | 1257  3061 | 1273  2773 | 1265
//   40000 of 33..50   1997 | 838   2016 | 851   1376 | 720   1311 | 727
// (With classes of 8, 16, 32 and 64 lanes in any order of sizes: 203 | 179,
// 73 | 80, 254 | 200, 83 | 79, 346 | 234, 840 | 411, 223 | 175, 1063 | 477,
// 3095 | 1283 and 2064 | 868.)  So: one class while the chip holds all but a
// few rounds of the problems at once, a wave each (its LDS holds 1024 of 64
// rows in FP64 and 2304 in FP32), and more the more problems there are.  The
// auction in FP64, whose problems take longer, has its classes from 3073
// problems on: 4000 of 2..8 rows 110 us (one class 161, classes of 8, 16, 32 and
// 64 lanes 152 with the bidding loop before), of 8..16 264 (434, 579), of 2..30
// 750 (633, 1358), of 2..64 2587 (1988, 5594).  With fewer problems one class
// loses less on narrow ranges than it gains on wide ones (2000 of 8..16 273 and
// 224 us, of 2..64 1779 and 2476), and it is below the 148 and 496 of before.
struct Classes {
    int count;
    int limit[5];   // largest size of each class, rising
};
inline Classes classes_for(int batch, int dtype, int solver)
{
    if (dtype == QAP_FP64)
        return batch <= (solver == QAP_LAP_SOLVER_AUCTION ? 3072 : 4096) ? Classes{1, {64}}
               : batch <= 8192                                          ? Classes{3, {16, 32, 64}}
                                                                        : Classes{5, {16, 32, 48, 56, 64}};
    return batch <= 8192    ? Classes{1, {64}}
           : batch <= 32768 ? Classes{3, {16, 32, 64}}
                            : Classes{4, {16, 32, 48, 64}};
}
// Up to this many problems all start at once, and their order does not matter.
constexpr int kUnsorted = 1024;

// Workspace of the device-side sort: kSortHeader ints (first place and number
// of problems of each class, the problems of each size and the places handed
// out of each size) followed by the `cap` problem indices in order.
constexpr int kSortHeader = 256;
constexpr int kSizes = QAP_RLT2_MAX_N + 1;
constexpr int kSizeCount = 64, kSizePlace = 160;   // first int of either in the header
static_assert(kSizeCount + kSizes <= kSizePlace && kSizePlace + kSizes <= kSortHeader, "header fields apart");

inline size_t sort_bytes(long long cap) { return (size_t)(kSortHeader + cap) * sizeof(int32_t); }

__global__ __launch_bounds__(kSortHeader) void k_sort_clear(int32_t* __restrict__ head) { head[threadIdx.x] = 0; }

// The problems by falling size, a counting sort (an unsolvable one sorts as the
// largest).  Each workgroup counts its problems by size in LDS, where the
// counting atomic is also a problem's rank among its workgroup's of that size.
// Up to kSortOne problems one workgroup does it all (PASS 0: no counters to
// clear, one launch); larger batches count in one launch (PASS 1) and write
// the list in a second one (PASS 2), with one global atomic per size and
// workgroup in each.  20000 problems took 16.5 us when every wave reserved its
// places class by class, and 13 in both passes now.  The order among
// problems of one size is not fixed; each problem's result depends only on its
// own matrix and the segment width, so it does not matter.
constexpr int kSortThreads = 1024, kSortEach = 4, kSortOne = kSortThreads * kSortEach;
template <int PASS>
__global__ __launch_bounds__(kSortThreads) void k_sort(int batch, const int32_t* __restrict__ n,
                                                       int32_t* __restrict__ head, int32_t* __restrict__ list,
                                                       Classes cl)
{
    __shared__ int cnt[kSizes], tot[kSizes], start[kSizes];
    const int t = threadIdx.x;
    if (t < kSizes) {
        cnt[t] = 0;
        tot[t] = PASS == 2 ? head[kSizeCount + t] : 0;
    }
    __syncthreads();
    int size[kSortEach], rank[kSortEach];
    const long long b0 = (long long)blockIdx.x * kSortOne + t;
#pragma unroll
    for (int u = 0; u < kSortEach; ++u) {
        const long long b = b0 + u * kSortThreads;
        size[u] = -1;
        if (b >= batch) continue;
        const int s = n[b];
        size[u] = s < 0 || s > QAP_RLT2_MAX_N ? QAP_RLT2_MAX_N : s;
    }
#pragma unroll
    for (int u = 0; u < kSortEach; ++u) rank[u] = size[u] >= 0 ? atomicAdd(&cnt[size[u]], 1) : 0;
    __syncthreads();
    if constexpr (PASS == 1) {
        if (t < kSizes && cnt[t] > 0) atomicAdd(&head[kSizeCount + t], cnt[t]);
        return;
    }
    if (t < kSizes) {
        // Problems of larger sizes come first.
        const int* all = PASS == 0 ? cnt : tot;
        int place = 0;
        for (int s = t + 1; s < kSizes; ++s) place += all[s];
        if (blockIdx.x == 0) {
            // A class starts with its largest size and ends with the size
            // above the next smaller class's.
            for (int c = 0; c < cl.count; ++c) {
                if (t == cl.limit[c]) head[2 * c] = place;
                if (t == (c > 0 ? cl.limit[c - 1] + 1 : 0)) {
                    int above = 0;   // larger sizes than the class's
                    for (int s = cl.limit[c] + 1; s < kSizes; ++s) above += all[s];
                    head[2 * c + 1] = place + all[t] - above;
                }
            }
        }
        if (PASS == 2 && cnt[t] > 0) place += atomicAdd(&head[kSizePlace + t], cnt[t]);
        start[t] = place;
    }
    __syncthreads();
#pragma unroll
    for (int u = 0; u < kSortEach; ++u)
        if (size[u] >= 0)
            list[start[size[u]] + rank[u]] = (int32_t)(b0 + u * kSortThreads);
}

// Largest batch of qap_lap_solve_noalloc: its work list is in the
// static array below, 4 MiB per device.
constexpr long long kNoAllocMaxBatch = QAP_LAP_NOALLOC_MAX_BATCH;

}  // namespace qap

// Work list of qap_lap_solve_noalloc, one copy on every device the
// library runs on, held until the process ends.  In host code this name is a
// host-side stand-in, not a device address: kernels and copies get the
// device address from hipGetSymbolAddress (scratch_address below).
static __device__ __align__(256) int32_t scratch[qap::kSortHeader + qap::kNoAllocMaxBatch];

namespace {

// Device address of `scratch` on the current device, looked up once per
// device (with that device current) and kept.
constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
void* g_scratch_addr[kMaxDevices] = {};

hipError_t scratch_address(int32_t** out)
{
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
    std::lock_guard<std::mutex> lock(g_scratch_mu);
    if (!g_scratch_addr[dev]) {
        void* p = nullptr;
        e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess) return e;
        g_scratch_addr[dev] = p;
    }
    *out = static_cast<int32_t*>(g_scratch_addr[dev]);
    return hipSuccess;
}

// The device-pointer solve, given a workspace of sort_bytes(batch) bytes (null
// up to kUnsorted problems): sort, then one launch per class with its grid
// sized for the whole batch (the kernel reads the class's range and idle
// waves exit), large problems first.
hipError_t solve_device(int batch, const int32_t* n, const int64_t* mat_off, const int64_t* vec_off, void* cost,
                        int dtype, double* value, void* duals, int32_t* assign, int wr, int solver, hipStream_t st,
                        int32_t* ws)
{
    const qap::Classes cl = qap::classes_for(batch, dtype, solver);
    if (!ws)
        return QAP_OPS(dtype, lap_batch(st, cl.limit[0], batch, nullptr, nullptr, n, mat_off, vec_off, cost, value,
                                        duals, assign, wr, solver));
    int32_t* list = ws + qap::kSortHeader;
    const dim3 threads(qap::kSortThreads);
    hipError_t e = hipSuccess;
    if (batch <= qap::kSortOne) {
        hipLaunchKernelGGL(qap::k_sort<0>, dim3(1), threads, 0, st, batch, n, ws, list, cl);
    } else {
        const dim3 grid((unsigned)(((long long)batch + qap::kSortOne - 1) / qap::kSortOne));
        hipLaunchKernelGGL(qap::k_sort_clear, dim3(1), dim3(qap::kSortHeader), 0, st, ws);
        if ((e = hipGetLastError()) != hipSuccess) return e;
        hipLaunchKernelGGL(qap::k_sort<1>, grid, threads, 0, st, batch, n, ws, list, cl);
        if ((e = hipGetLastError()) != hipSuccess) return e;
        hipLaunchKernelGGL(qap::k_sort<2>, grid, threads, 0, st, batch, n, ws, list, cl);
    }
    if ((e = hipGetLastError()) != hipSuccess) return e;
    for (int c = cl.count - 1; c >= 0; --c) {
        e = QAP_OPS(dtype, lap_batch(st, cl.limit[c], batch, ws + 2 * c, list, n, mat_off, vec_off, cost, value, duals,
                                     assign, wr, solver));
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

qap_status check_common(int batch, const int32_t* n, const int64_t* mat_off, const int64_t* vec_off,
                        const void* cost, int dtype, const double* value, const void* duals, const int32_t* assign)
{
    if (batch < 0) return fail(QAP_EINVAL, "negative batch");
    if (batch == 0) return QAP_OK;
    if (!n || !mat_off || !cost || !value) return fail(QAP_EINVAL, "null n, mat_off, cost or value");
    if ((duals || assign) && !vec_off) return fail(QAP_EINVAL, "vec_off needed for duals or assign");
    if (dtype != QAP_FP64 && dtype != QAP_FP32_CERTIFIED && dtype != QAP_FP32_NEAREST)
        return fail(QAP_EINVAL, "unknown dtype");
    return QAP_OK;
}

}  // namespace

extern "C" {

qap_status qap_lap_solve(int batch, const int32_t* n, const int64_t* mat_off, const int64_t* vec_off, void* cost,
                         int dtype, double* value, void* duals, int32_t* assign, int flags, void* stream)
{
    qap::last_error().clear();
    qap_status cs = check_common(batch, n, mat_off, vec_off, cost, dtype, value, duals, assign);
    if (cs != QAP_OK || batch == 0) return cs;
    const size_t es = dtype == QAP_FP64 ? sizeof(double) : sizeof(float);
    hipStream_t st = static_cast<hipStream_t>(stream);
    const int wr = (flags & QAP_LAP_RESIDUAL) ? 1 : 0;
    const int solver = (flags & QAP_LAP_AUCTION) ? QAP_LAP_SOLVER_AUCTION : QAP_LAP_SOLVER_CANONICAL;
    if (flags & QAP_LAP_DEVICE) {
        // The work list's memory comes from the stream-ordered allocator, so
        // the call stays asynchronous and calls on other streams get their own.
        void* ws = nullptr;
        hipError_t e = batch > qap::kUnsorted ? hipMallocAsync(&ws, qap::sort_bytes(batch), st) : hipSuccess;
        if (e == hipErrorOutOfMemory && qap::give_back_kept_memory())
            e = hipMallocAsync(&ws, qap::sort_bytes(batch), st);
        if (e != hipSuccess)
            return fail(e == hipErrorOutOfMemory ? QAP_ENOMEM : QAP_EDEVICE,
                        std::string("hipMallocAsync: ") + hipGetErrorString(e));
        e = solve_device(batch, n, mat_off, vec_off, cost, dtype, value, duals, assign, wr, solver, st,
                         static_cast<int32_t*>(ws));
        const hipError_t ef = ws ? hipFreeAsync(ws, st) : hipSuccess;
        if (e != hipSuccess) return fail(QAP_EDEVICE, std::string("kernel launch: ") + hipGetErrorString(e));
        if (ef != hipSuccess) return fail(QAP_EDEVICE, std::string("hipFreeAsync: ") + hipGetErrorString(ef));
        return QAP_OK;
    }
    // Host pointers: validate, sort by size, stage, solve, copy back.
    int64_t mat_end = 0, vec_end = 0;
    std::vector<int32_t> idx(batch);   // problems by falling size
    for (int b = 0; b < batch; ++b) {
        if (n[b] < 0 || n[b] > QAP_RLT2_MAX_N) return fail(QAP_EINVAL, "n[b] must be in [0, 64]");
        if (mat_off[b] < 0) return fail(QAP_EINVAL, "negative mat_off");
        mat_end = std::max(mat_end, mat_off[b] + (int64_t)n[b] * n[b]);
        for (int64_t e = 0; e < (int64_t)n[b] * n[b]; ++e) {
            const double x = dtype == QAP_FP64 ? static_cast<const double*>(cost)[mat_off[b] + e]
                                               : (double)static_cast<const float*>(cost)[mat_off[b] + e];
            if (!std::isfinite(x)) return fail(QAP_EINVAL, "non-finite cost entry");
        }
        if (vec_off) {
            if (vec_off[b] < 0) return fail(QAP_EINVAL, "negative vec_off");
            vec_end = std::max(vec_end, vec_off[b] + (int64_t)n[b]);
        }
        idx[b] = b;
    }
    std::stable_sort(idx.begin(), idx.end(), [n](int32_t x, int32_t y) { return n[x] > n[y]; });
    int32_t *dn = nullptr, *didx = nullptr;
    int64_t *dmo = nullptr, *dvo = nullptr;
    void *dcost = nullptr, *ddual = nullptr;
    double* dval = nullptr;
    int32_t* dassign = nullptr;
    qap_status result = QAP_OK;
    auto cleanup = [&]() {
        for (void* p : {(void*)dn, (void*)didx, (void*)dmo, (void*)dvo, (void*)dcost, (void*)dval, (void*)ddual,
                        (void*)dassign})
            if (p) (void)hipFree(p);
    };
#define CK2(call)                                                                                    \
    do {                                                                                             \
        hipError_t e_ = (call);                                                                      \
        if (e_ != hipSuccess) {                                                                      \
            result = fail(e_ == hipErrorOutOfMemory ? QAP_ENOMEM : QAP_EDEVICE,                      \
                          std::string(#call) + ": " + hipGetErrorString(e_));                        \
            cleanup();                                                                               \
            return result;                                                                           \
        }                                                                                            \
    } while (0)
    CK2(qap::device_malloc(&dn, batch * sizeof(int32_t)));
    CK2(qap::device_malloc(&didx, batch * sizeof(int32_t)));
    CK2(qap::device_malloc(&dmo, batch * sizeof(int64_t)));
    CK2(qap::device_malloc(&dcost, std::max<int64_t>(mat_end, 1) * es));
    CK2(qap::device_malloc(&dval, batch * sizeof(double)));
    CK2(hipMemcpyAsync(dn, n, batch * sizeof(int32_t), hipMemcpyHostToDevice, st));
    CK2(hipMemcpyAsync(didx, idx.data(), batch * sizeof(int32_t), hipMemcpyHostToDevice, st));
    CK2(hipMemcpyAsync(dmo, mat_off, batch * sizeof(int64_t), hipMemcpyHostToDevice, st));
    if (mat_end > 0) CK2(hipMemcpyAsync(dcost, cost, mat_end * es, hipMemcpyHostToDevice, st));
    if (vec_off) {
        CK2(qap::device_malloc(&dvo, batch * sizeof(int64_t)));
        CK2(hipMemcpyAsync(dvo, vec_off, batch * sizeof(int64_t), hipMemcpyHostToDevice, st));
    }
    if (duals) CK2(qap::device_malloc(&ddual, std::max<int64_t>(4 * vec_end, 1) * es));
    if (assign) CK2(qap::device_malloc(&dassign, std::max<int64_t>(vec_end, 1) * sizeof(int32_t)));
    // One launch per size class, of the width and LDS of its largest problem
    // (the table above is for launches that do not know it).  4000 problems of
    // 30 rows by the auction took 12.9 ms in all with LDS for 64 rows and a wave
    // each, 11.6 now; the canonical solve, whose time is mostly the copies', 10.5
    // either way.
    const qap::Classes cl = qap::classes_for(batch, dtype, solver);
    int first = 0;
    for (int c = cl.count - 1; c >= 0; --c) {
        int end = first;
        while (end < batch && (c == 0 || n[idx[end]] > cl.limit[c - 1])) ++end;
        if (end > first)
            CK2(QAP_OPS(dtype, lap_batch(st, std::max(16, n[idx[first]]), end - first, nullptr, didx + first, dn, dmo, dvo, dcost, dval,
                                         ddual, dassign, wr, solver)));
        first = end;
    }
    CK2(hipMemcpyAsync(value, dval, batch * sizeof(double), hipMemcpyDeviceToHost, st));
    if (wr && mat_end > 0) CK2(hipMemcpyAsync(cost, dcost, mat_end * es, hipMemcpyDeviceToHost, st));
    if (duals && vec_end > 0) CK2(hipMemcpyAsync(duals, ddual, 4 * vec_end * es, hipMemcpyDeviceToHost, st));
    if (assign && vec_end > 0)
        CK2(hipMemcpyAsync(assign, dassign, vec_end * sizeof(int32_t), hipMemcpyDeviceToHost, st));
    CK2(hipStreamSynchronize(st));
#undef CK2
    cleanup();
    return QAP_OK;
}

qap_status qap_lap_solve_noalloc(int batch, const int32_t* n, const int64_t* mat_off, const int64_t* vec_off,
                                 void* cost, int dtype, double* value, void* duals, int32_t* assign, int flags,
                                 void* stream)
{
    qap::last_error().clear();
    qap_status cs = check_common(batch, n, mat_off, vec_off, cost, dtype, value, duals, assign);
    if (cs != QAP_OK || batch == 0) return cs;
    if (!(flags & QAP_LAP_DEVICE))
        return fail(QAP_EINVAL, "qap_lap_solve_noalloc takes device pointers only (flags must hold QAP_LAP_DEVICE)");
    if (batch > qap::kNoAllocMaxBatch)
        return fail(QAP_EINVAL, "batch exceeds QAP_LAP_NOALLOC_MAX_BATCH (" +
                                    std::to_string(qap::kNoAllocMaxBatch) + ") problems");
    int32_t* ws = nullptr;
    hipError_t e = batch > qap::kUnsorted ? scratch_address(&ws) : hipSuccess;
    if (e != hipSuccess) return fail(QAP_EDEVICE, std::string("hipGetSymbolAddress: ") + hipGetErrorString(e));
    e = solve_device(batch, n, mat_off, vec_off, cost, dtype, value, duals, assign,
                     (flags & QAP_LAP_RESIDUAL) ? 1 : 0,
                     (flags & QAP_LAP_AUCTION) ? QAP_LAP_SOLVER_AUCTION : QAP_LAP_SOLVER_CANONICAL,
                     static_cast<hipStream_t>(stream), ws);
    if (e != hipSuccess) return fail(QAP_EDEVICE, std::string("kernel launch: ") + hipGetErrorString(e));
    return QAP_OK;
}

}  // extern "C"
