// Cost-concentration kernels (Section 4.1 of arXiv 1510.02065).  Each wave
// works on 64/SEG assignment problems at once (one per SEG-lane segment), each
// staged in the wave's own LDS region; a workgroup is one wave.  Problems of
// every instance of a handle are served by one launch per segment-size class.
#pragma once
#include "lap_auction.hpp"
#include "lap_slots.hpp"
#include "lap_wave.hpp"

namespace qap {

// Problems of a family, for the instances of one segment-size class:
// cls[0..Kc) are the instance ids and pre[] the prefix sums of their problem
// counts, so problem x belongs to instance cls[find_seg(pre, Kc, x)].  A launch
// of k_lap_family_s takes the problems from `first` on.
struct FamilyClass {
    const int* cls;
    const long long* pre;
    int Kc;
    long long total;
    long long first;
};

enum LapFamily : int { kFamD = 0, kFamC = 1 };

// How the D family is stored and enumerated (see pair_block).
enum DStorage : int {
    kAllBlocks = 0,    // every block stored (block-major); problem b is block b, parent c_b
    kHalfStore = 1     // one block per complementary pair stored (pair-major);
                       // problem h is stored block h, parents c_beta and c_twin
};

// Copy an n x n block (rows `rows` in global memory) into LDS (row stride
// ldm).  Each lane issues the loads of a whole chunk of rows before it writes
// any of them, so a wave waits for HBM once per chunk instead of once per row:
// the first 24 rows (16 and 8 for the segments of that width, which hold no
// more; with 24 in all of them N = 18 took 83.2 us for step 4, now 81.4) in
// straight-line code, the rest kStageTail at a time.  Rows past the end re-read row n-1 and write
// it again (the same value to the same place), so no write is guarded.  Row
// offsets in LDS are 24-bit products; those in global memory stay below 2^32
// bytes (a row stride is at most N (N-1) (N-2) < 2^18 entries for N <= 64).
template <int SEG>
constexpr int kStageRows = SEG < 24 ? SEG : 24;
constexpr int kStageTail = 8;

template <typename T, int SEG, typename Rows>
__device__ __forceinline__ void stage_block(T* __restrict__ M, int ldm, const Rows& rows, int n, int c)
{
    if (c >= n) return;
    {
        T t[kStageRows<SEG>];
#pragma unroll
        for (int u = 0; u < kStageRows<SEG>; ++u) t[u] = rows.at(min(u, n - 1));
#pragma unroll
        for (int u = 0; u < kStageRows<SEG>; ++u) M[__umul24((unsigned)min(u, n - 1), (unsigned)ldm) + c] = t[u];
    }
    if constexpr (SEG > kStageRows<SEG>) {
        for (int r0 = kStageRows<SEG>; r0 < n; r0 += kStageTail) {
            T t[kStageTail];
#pragma unroll
            for (int u = 0; u < kStageTail; ++u) t[u] = rows.at(min(r0 + u, n - 1));
#pragma unroll
            for (int u = 0; u < kStageTail; ++u) M[__umul24((unsigned)min(r0 + u, n - 1), (unsigned)ldm) + c] = t[u];
        }
    }
}

// Stage one problem per segment and solve it (the residual written over the
// block where `active`); S to every lane.  UNI: the size is a scalar, as when
// every problem of the wave belongs to one instance, so that loop counts,
// clamps, bit masks and LDS offsets that depend only on n run on the scalar
// unit; otherwise it is a lane's (a wave across an instance boundary, or with
// segments past the last problem, whose n is 0).  Both compute the same values.
template <typename T, int SEG, bool AUC, bool DOWN, bool UNI, typename Rows>
__device__ __forceinline__ double stage_and_solve(unsigned char* smem, int seg, int lane, int nmax, int n,
                                                  const Rows& rows, bool active, int32_t* assign = nullptr)
{
    const LapScratch<T> sc(smem + seg * LapLds<T, AUC>::bytes(nmax), n);
    stage_block<T, SEG>(sc.M, sc.ld, rows, n, lane);
    wave_sync();
    T* const no_duals = nullptr;
    if constexpr (AUC)
        return lap_auction_flat<T, SEG, DOWN>(sc, n, rows, active, no_duals, assign);
    else
        return lap_concentrate<T, SEG, DOWN, UNI>(sc, n, rows, active, no_duals, assign);
}

// D -> C (FAM kFamD: blocks D_beta of size N-2, parent c_beta) or C -> B
// (kFamC: blocks C_ij of size N-1, parent b_ij), one column per lane, 64/SEG
// problems per wave, one wave per workgroup.  parent += S, the block is
// replaced by its residual, values[...] = S when values is not null (values
// are packed like the parents).  `mode` applies to the D family only.  AUC:
// the auction solver.  Registers: the FP32 kernels are held to 72 VGPRs (seven
// waves per SIMD; held to 64, eight waves, they spill 11 and N = 25 took 474
// against 462 us) and the FP64 ones of up to 32 lanes to 80 (six waves; with
// 96, five waves, N = 20 took 219 against 208 us and N = 25 the same).
//
// What bounds it is the chain of dependent instructions of each wave, at as
// many waves as LDS admits; FP32 and small sizes are also close to the VALU's
// rate, so work that a wave has in common goes to the scalar unit.  All
// problems of a wave belong to one instance except where it crosses into the
// next (every wave of a single instance but the last, all but one wave per
// instance of a batch): such a wave finds its instance, its rows' addresses
// and its loop counts with scalar instructions (N = 25 FP32 468 -> 448 us, N =
// 33 2720 -> 2612; a batch of 160 nodes of N = 10..22 52.3 -> 50.2 ms).
template <int PM, int SEG, int FAM, bool AUC = false>
__global__ __launch_bounds__(64, PM != kPrecF64 ? 7 : (SEG <= 32 ? 6 : 1))
void k_lap_family_s(StoreT<PM>* __restrict__ D, StoreT<PM>* __restrict__ C, StoreT<PM>* __restrict__ B,
                    const Inst* __restrict__ inst, FamilyClass fc, int nmax, double* __restrict__ values, int mode,
                    const int* __restrict__ act)
{
    using T = StoreT<PM>;
    constexpr bool DOWN = PM == kPrecF32Down;
    extern __shared__ __align__(16) unsigned char smem[];
    constexpr int LPW = 64 / SEG;
    const int seg = threadIdx.x / SEG;
    const int lane = threadIdx.x & (SEG - 1);
    T* __restrict__ const parent = (FAM == kFamD) ? C : B;
    // Problem b of instance I: size, offset of its block in D (C), row stride
    // in entries, and this lane's parent at up + p (lane 0 has the first,
    // lane 1 the twin's; p < 0: none).
    struct Problem {
        int n;
        long long off, ld, up;
        int p;
    };
    const int only = lane == 0 ? 0 : -1;
    auto problem = [&](const Inst& I, long long b) __attribute__((always_inline)) -> Problem {
        if constexpr (FAM == kFamD) {
            const int n = I.N - 2;
            if (mode == kAllBlocks) return {n, I.offD + b * I.ldD, n, I.offC, (int)b | only};
            long long beta, twin, first;
            pair_block(I.N, b, &beta, &twin, &first);
            return {n, I.offD + first, (long long)I.N * (I.N - 1) * n, I.offC,
                    lane == 0 ? (int)beta : lane == 1 ? (int)twin : -1};
        } else {
            const int n = I.N - 1;
            return {n, I.offC + b * (long long)(n * n), n, I.offB, (int)b | only};
        }
    };
    T* const blocks = FAM == kFamD ? D : C;
    auto finish = [&](const Problem& q, T par, double S) __attribute__((always_inline)) {
        if (q.p < 0) return;
        (parent + q.up)[q.p] = store_add<PM>(par, S);
        if (values) (values + q.up)[q.p] = S;
    };
    // The parents are read before the solve, so that the wave does not wait
    // for them at its end.
    const long long x0 = fc.first + xcd_major(blockIdx.x, gridDim.x) * LPW;
    const int k0 = find_seg(fc.pre, fc.Kc, x0);
    const int id0 = fc.cls[k0];
    const long long end0 = k0 + 1 < fc.Kc ? fc.pre[k0 + 1] : fc.total;
    if (x0 + LPW <= end0) {
        // Every problem of the wave belongs to instance id0; its blocks lie at
        // growing offsets, less than 2^32 bytes apart (a facility pair's
        // stored rows are below 2^27).
        if (!act[id0]) return;
        const Inst I = inst[id0];
        const Problem q = problem(I, x0 - fc.pre[k0] + seg);
        const T par = q.p >= 0 ? (parent + q.up)[q.p] : (T)0;
        const unsigned lo = (unsigned)__builtin_amdgcn_readfirstlane((int)(unsigned)q.off);
        const unsigned hi = (unsigned)__builtin_amdgcn_readfirstlane((int)(unsigned)(q.off >> 32));
        const long long first = (long long)(((unsigned long long)hi << 32) | lo);
        const int n = FAM == kFamD ? I.N - 2 : I.N - 1;
        const unsigned ld = FAM == kFamD && mode != kAllBlocks ? (unsigned)(I.N * (I.N - 1) * n) : (unsigned)n;
        const WaveRows<T> rows{reinterpret_cast<char*>(blocks + first), ld * (unsigned)sizeof(T),
                               (unsigned)(q.off - first + lane) * (unsigned)sizeof(T)};
        const double S = stage_and_solve<T, SEG, AUC, DOWN, true>(smem, seg, lane, nmax, n, rows, true);
        finish(q, par, S);
        return;
    }
    const long long x = x0 + seg;
    int kk = 0;
    if (x < fc.total) kk = find_seg(fc.pre, fc.Kc, x);
    const bool active = x < fc.total && act[fc.cls[kk]];
    Problem q{0, 0, 0, 0, -1};
    T par = 0;
    if (active) {
        q = problem(inst[fc.cls[kk]], x - fc.pre[kk]);
        if (q.p >= 0) par = (parent + q.up)[q.p];
    }
    const LaneRows<T> rows{blocks + q.off + lane, q.ld};
    const double S = stage_and_solve<T, SEG, AUC, DOWN, false>(smem, seg, lane, nmax, q.n, rows, active);
    if (active) finish(q, par, S);
}

// B -> LB' and LB += LB' (steps 7-8), one problem of size N per instance of
// the class.  lb[2k] = LB, lb[2k+1] = LB' (FP64; in FP32
// certified mode the bound accumulates rounding toward -inf).  The instance's
// trace gets (LB, LB') at position t = counter[k]++ when below trace_cap
// (entry t of the handle's `count` instances next to each other), and
// sigma (nullable, packed like B) the assignment of the B problem, a
// permutation of the instance.  Stop rule of Algorithm 1, with stop[0] = K and
// stop[1] = UB (UB <= 0: none): the instance's act flag is cleared once
// LB >= UB or LB' / UB < K.
template <int PM, int SEG, bool AUC = false>
__global__ __launch_bounds__(64) void k_lap_B_s(StoreT<PM>* __restrict__ B, const Inst* __restrict__ inst,
                                                FamilyClass fc, int nmax, double* __restrict__ lb,
                                                double* __restrict__ trace, long long* __restrict__ counter,
                                                long long trace_cap, int count, double* __restrict__ values,
                                                int32_t* __restrict__ sigma, int* __restrict__ act,
                                                const double* __restrict__ stop)
{
    using T = StoreT<PM>;
    constexpr bool DOWN = PM == kPrecF32Down;
    extern __shared__ __align__(16) unsigned char smem[];
    constexpr int LPW = 64 / SEG;
    const int seg = threadIdx.x / SEG;
    const int lane = threadIdx.x & (SEG - 1);
    const long long x = (long long)blockIdx.x * LPW + seg;
    const int k = x < fc.total ? fc.cls[x] : 0;
    const bool active = x < fc.total && act[k];
    const Inst I = inst[k];
    const int n = active ? I.N : 0;
    T* blk = B + I.offB;
    int32_t* sg = (active && sigma) ? sigma + I.offB : nullptr;
    const LaneRows<T> rows{blk + lane, n};
    const int nu = __builtin_amdgcn_readfirstlane(n);
    const double S = ballot64(n != nu) == 0
                         ? stage_and_solve<T, SEG, AUC, DOWN, true>(smem, seg, lane, nmax, nu, rows, active, sg)
                         : stage_and_solve<T, SEG, AUC, DOWN, false>(smem, seg, lane, nmax, n, rows, active, sg);
    if (active && lane == 0) {
        const double L = DOWN ? add_down(lb[2 * k], S) : lb[2 * k] + S;
        lb[2 * k] = L;
        lb[2 * k + 1] = S;
        if (values) values[k] = S;
        if (counter) {
            const long long t = counter[k];
            if (trace && t < trace_cap) {
                trace[(t * count + k) * 2] = L;
                trace[(t * count + k) * 2 + 1] = S;
            }
            counter[k] = t + 1;
        }
        const double Kp = stop[0], UB = stop[1];
        if (UB > 0.0 && (L >= UB || (Kp > 0.0 && S < Kp * UB))) act[k] = 0;
    }
}

// Generic batch (qap_lap_solve), workgroups from `first` on: slot s < count
// solves problem
// b = idx[r + s] (b = s when idx is null).  With `range` (device memory) r =
// range[0] and count = range[1]; without it they are 0 and `count`.  Problem b
// has size n[b] (<= nmax <= SEG, else its value is NaN and nothing else is written), matrix at
// cost + mat_off[b], vectors at vec_off[b] (vec_off may be null when duals and
// assign are).  The launch's LDS holds problems of up to nmax.  AUC: the
// auction solver (lap_auction_flat) instead of the canonical dual.
template <int PM, int SEG, bool AUC>
__global__ __launch_bounds__(64) void k_lap_batch(long long first, int count, const int* __restrict__ range,
                                                  const int32_t* __restrict__ idx, int nmax,
                                                  const int32_t* __restrict__ nv,
                                                  const int64_t* __restrict__ mat_off,
                                                  const int64_t* __restrict__ vec_off,
                                                  StoreT<PM>* __restrict__ cost, double* __restrict__ value,
                                                  StoreT<PM>* __restrict__ duals, int32_t* __restrict__ assign,
                                                  int write_residual)
{
    using T = StoreT<PM>;
    extern __shared__ __align__(16) unsigned char smem[];
    constexpr int LPW = 64 / SEG;
    const int seg = threadIdx.x / SEG;
    const int lane = threadIdx.x & (SEG - 1);
    const int cnt = range ? range[1] : count;
    const int64_t s0 = (first + blockIdx.x) * LPW, s = s0 + seg;
    if (s0 >= cnt) return;
    const bool in = s < cnt;
    const int64_t b = !in ? 0 : idx ? (int64_t)idx[(range ? range[0] : 0) + s] : s;
    int n = in ? nv[b] : 0;
    const bool bad = n < 0 || n > nmax;
    if (bad) n = 0;
    T* const mat = n > 0 ? cost + mat_off[b] : cost;
    const int64_t vo = (n > 0 && vec_off) ? vec_off[b] : 0;
    const bool wr = write_residual && n > 0;
    T* const dw = (duals && n > 0) ? duals + 4 * vo : nullptr;
    int32_t* const aw = (assign && n > 0) ? assign + vo : nullptr;
    // The size as a scalar when every problem of the wave has it.
    auto solve = [&](int nn, auto uni) __attribute__((always_inline)) -> double {
        const LapScratch<T> sc(smem + seg * LapLds<T, AUC>::bytes(nmax), nn);
        const LaneRows<T> rows{mat + lane, nn};
        stage_block<T, SEG>(sc.M, sc.ld, rows, nn, lane);
        wave_sync();
        if constexpr (AUC)
            return lap_auction_flat<T, SEG, PM == kPrecF32Down>(sc, nn, rows, wr, dw, aw);
        else
            return lap_concentrate<T, SEG, PM == kPrecF32Down, decltype(uni)::value>(sc, nn, rows, wr, dw, aw);
    };
    const int nu = __builtin_amdgcn_readfirstlane(n);
    const double S = ballot64(n != nu) == 0 ? solve(nu, std::true_type{}) : solve(n, std::false_type{});
    // A quiet NaN written by bit pattern marks a problem that was not solved.
    if (in && lane == 0) value[b] = bad ? __longlong_as_double(0x7ff8000000000000ll) : S;
}

}  // namespace qap
