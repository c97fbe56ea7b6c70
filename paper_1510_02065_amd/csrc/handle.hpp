// Internal host-side state of a qap_rlt2 handle, shared by the C ABI
// (api.hip) and the per-precision launch code (ops_*.hip).
#pragma once
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstring>
#include <string>
#include <vector>

#include "inherit_kernels.hpp"
#include "qap_rlt2.h"

namespace qap {

// Thread-local message of the last failure (qap_last_error).
std::string& last_error();

inline qap_status fail(qap_status st, const std::string& msg)
{
    last_error() = msg;
    return st;
}

#define QAP_HIP(call)                                                                          \
    do {                                                                                       \
        hipError_t e_ = (call);                                                                \
        if (e_ != hipSuccess)                                                                  \
            return ::qap::fail(QAP_EDEVICE, std::string(#call) + ": " + hipGetErrorString(e_)); \
    } while (0)

inline int seg_for(int n)
{
    if (n <= 8) return 8;
    if (n <= 16) return 16;
    if (n <= 32) return 32;
    return 64;
}

// Workgroups for `work` items, `each` of them per workgroup.
inline long long groups_of(long long work, int each) { return (work + each - 1) / each; }

// A launch has fewer than 2^32 threads (their number is taken modulo that: the
// rest does not run, and there is no error).  f(first, count) launches
// workgroups first .. first + count - 1 of `groups` and returns its error; it is
// called as often as that takes (once for all but the largest batches).
template <typename F>
hipError_t in_launches(long long groups, int threads, F f)
{
    const long long most = 0xffffffffll / threads / 8 * 8;
    hipError_t e = hipSuccess;
    for (long long first = 0; first < groups && e == hipSuccess; first += most)
        e = f(first, (unsigned)(groups - first < most ? groups - first : most));
    return e;
}

// Per-instance trace entries kept on the device between host reads, and the
// rows of the device's trace: besides those, entries already read.
constexpr long long kTraceCap = 1024, kTraceSlack = 64, kTraceRows = kTraceCap + kTraceSlack;

// LDS of a one-wave workgroup of the assignment kernels at size nmax.
template <typename T, int SEG, bool AUC>
size_t slot_lds(int nmax) { return (size_t)(64 / SEG) * LapLds<T, AUC>::bytes(nmax); }

// Instances of one family that share a segment size.
struct ClassHost {
    int seg = 0;       // lanes per problem: next power of two >= n (8 at least)
    int nmax = 0;
    std::vector<int> ids;
    std::vector<long long> pre;
    long long total = 0;
    int* d_ids = nullptr;
    long long* d_pre = nullptr;
    FamilyClass dev(long long first) const { return FamilyClass{d_ids, d_pre, (int)ids.size(), total, first}; }
};

// Instances of one size: steps 1-3 run one launch per size, with the kernel,
// the workgroup width and the LDS for that size, so a CU holds as many of the
// small instances' workgroups as fit.
constexpr int kSweepBox = -1;
struct SweepClass {
    int N = 0;
    std::vector<int> ids;          // instances of this size
    std::vector<long long> pre;    // first workgroup of each, within the launch (kSweepBox), or first triple
    long long nwg = 0;             // workgroups (kSweepBox) or triples of the launch
    int nt = 0;                    // threads of a per-triple workgroup, 0: persistent kernel, kSweepBox: k_sweep_box
    int* d_ids = nullptr;
    long long* d_pre = nullptr;
};

}  // namespace qap

struct qap_rlt2 {
    int K = 0;
    int precision = QAP_FP64;
    int level = 2;                 // 2: RLT2 (B, C, D); 1: RLT1 (B, C only)
    int device = 0;
    hipStream_t stream = nullptr;
    bool own_stream = false;
    int trace_level = 1;
    int use_graph = 1;
    int lap_solver = QAP_LAP_SOLVER_CANONICAL;   // qap_lap_solver of the concentrations
    long long pending = 0;   // iterations of qap_rlt2_step whose trace entries are still on the device
    int dmode = qap::kHalfStore;   // D storage and enumeration (kAllBlocks or kHalfStore)
    int Nmax = 0;                  // largest instance
    size_t lds_limit = 65536;   // dynamic LDS a workgroup may request
    int num_cu = 256;           // compute units of the device
    size_t elem = 8;   // bytes per reduced cost
    size_t bytesD = 0;   // of D
    size_t allocD = 0;   // of the allocation it is in
    double stopK = 0.0, stopUB = 0.0;   // stop rule of Algorithm 1 (UB <= 0: off)
    std::vector<qap::Inst> inst;
    long long totalB = 0, totalC = 0, totalD = 0, totalWG = 0;
    std::vector<long long> preB, preC, preWG;
    std::vector<long long> preP;      // first facility pair of each instance
    long long totalP = 0;
    std::vector<long long> preCert;   // first k_cert_pairs workgroup of each instance
    long long totalCert = 0;
    qap::ClassHost fam[3][4];   // [D, C, B][segment class]
    std::vector<qap::SweepClass> sweep_cls;   // kHalfStore: one sweep launch per instance size, largest first
    // Overlapped steps 1-4 of a batch of mixed sizes (qap_rlt2_ascend): the
    // sweep of each size runs on `stream`, and the D->C concentration of that
    // size on `stream2` as soon as its sweep is done, so one size's
    // assignment problems run beside the next size's sweep.
    bool overlap = false;
    hipStream_t stream2 = nullptr;
    std::vector<qap::ClassHost> famD_size;    // D family of each sweep class's instances (same order)
    std::vector<hipEvent_t> ev_size;          // one per sweep class: its sweep is done
    hipEvent_t ev_fork = nullptr, ev_join = nullptr;
    std::vector<int> tri;                     // facility triples of every instance
    void* arena = nullptr;   // every device array below but D, dCt and dBt
    qap::Inst* dInst = nullptr;
    long long *dPreB = nullptr, *dPreC = nullptr, *dPreWG = nullptr, *dPreCert = nullptr, *dPreP = nullptr;
    void* dB = nullptr;
    void* dC = nullptr;
    void* dD = nullptr;
    void* dCC = nullptr;
    double *dF = nullptr, *dDm = nullptr, *dB0 = nullptr;   // the instances' data, N^2 entries each
    int* dFix = nullptr;        // a children handle's (facility, location) pairs
    double* dLB = nullptr;      // [LB, LB'] per instance
    double* dValD = nullptr;    // per-block values of the last step 4 (packed like C)
    double* dValC = nullptr;    // per-block values of the last step 6 (packed like B)
    double* dValB = nullptr;    // per-instance value of the last step 7
    // One record, read back in one copy: dCounter (K), dLB (2 K), dTrace.
    double* dTrace = nullptr;   // kTraceRows x K x (LB, LB')
    long long* dCounter = nullptr;   // trace entries of each instance
    std::vector<long long> seen;     // those of them already read back
    int* dTri = nullptr;
    int* dAct = nullptr;        // per-instance flag: the dual ascent still runs
    double* dStop = nullptr;    // (K, UB) of the stop rule
    int32_t* dSigma = nullptr;  // assignment of the last B problem (packed like B)
    double* dCt = nullptr;      // certification: c~ (packed like C), allocated by the first certification
    double* dBt = nullptr;      // certification: b~ (packed like B)
    double* dCert = nullptr;    // certification result per instance
    hipGraphExec_t graph_exec = nullptr;   // kGraphIters iterations
    int64_t launched = 0;                  // iterations enqueued by qap_rlt2_ascend
    hipGraph_t graph = nullptr;
    std::vector<std::vector<double>> tLB, tLBp;
    std::vector<int64_t> itk;       // loop iterations each instance has run
    bool broken = false;
};

namespace qap {

// Free the memory kept on the current device for later handles (after a failed
// allocation); whether there was any.
bool give_back_kept_memory();

// hipMalloc, tried again without the kept memory when it fails for space.
template <typename X>
hipError_t device_malloc(X** p, size_t bytes)
{
    hipError_t e = hipMalloc(p, bytes);
    if (e == hipErrorOutOfMemory && give_back_kept_memory()) e = hipMalloc(p, bytes);
    return e;
}

// Launch code of one precision mode (ops_impl.hpp, instantiated in
// ops_f64.hip, ops_f32d.hip and ops_f32n.hip).
template <int PM>
struct Ops {
    // One step of an iteration: 3 (steps 1-3, or step 1 at level 1), 4, 5,
    // 6, 7 (steps 7-8).
    static hipError_t enqueue_step(qap_rlt2* h, int step);
    // Steps 1 and 5 of a level-1 iteration (3 and 5 of enqueue_step).
    static hipError_t enqueue_spread_transfer(qap_rlt2* h);
    // FP64 certification cascade into h->dCert.
    static hipError_t certify(qap_rlt2* h);
    // Initial dual of instance k from device copies of F, D and B0 (nullable).
    static hipError_t init_instance(qap_rlt2* h, int k, const double* dF, const double* dDm, const double* dB0);
    // Kernel of steps 1-3 at size N (SweepClass::nt).
    static int sweep_threads(int N, size_t lds_limit);
    // Location tiles per axis of k_sweep_box at size N.
    static int sweep_tiles(int N);
    // Batched assignment problems (qap_lap_solve) of sizes up to nmax (at
    // least 16): the first `count` (of idx when it is not null) or, with
    // `range` in device memory, the range[1] (at most `count`) from
    // idx[range[0]] on, by the canonical dual or the auction (solver, a qap_lap_solver value).
    static hipError_t lap_batch(hipStream_t st, int nmax, int count, const int* range, const int32_t* idx,
                                const int32_t* n, const int64_t* mo, const int64_t* vo, void* cost, double* value,
                                void* duals, int32_t* assign, int wr, int solver);
    // Children of parent instance pk of handle ph (fixings fix[2c], fix[2c+1]
    // in device memory) into handle ch, whose instances are those children.
    static hipError_t inherit(qap_rlt2* ph, int pk, qap_rlt2* ch, const int* dfix);
    // Steps 1-4 with each size's concentration overlapped with the next
    // size's sweep (h->overlap).
    static hipError_t enqueue_sweep_concentrate_overlapped(qap_rlt2* h);
};

extern template struct Ops<kPrecF64>;
extern template struct Ops<kPrecF32Down>;
extern template struct Ops<kPrecF32Near>;

// Dispatch to Ops<precision>.
#define QAP_OPS(prec, call)                                     \
    ((prec) == ::qap::kPrecF64       ? ::qap::Ops<::qap::kPrecF64>::call      \
     : (prec) == ::qap::kPrecF32Down ? ::qap::Ops<::qap::kPrecF32Down>::call  \
                                     : ::qap::Ops<::qap::kPrecF32Near>::call)

}  // namespace qap
