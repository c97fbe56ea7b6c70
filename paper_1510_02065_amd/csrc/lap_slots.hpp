// Linear assignment with canonical dual on gfx950: the solver of every
// assignment kernel (the concentrations and the batched qap_lap_solve).
//
// Cost concentration (Section 4.1 of arXiv 1510.02065) solves one assignment
// problem per block of the reduced-cost array, moves its value S to the
// parent coefficient and replaces the block by its residuals.  Here a segment
// of SEG lanes owns one n x n problem (n <= SEG) whose matrix sits in LDS;
// lane l holds column l (and, in the row passes, row l).  A wave carries
// 64/SEG problems.
//
// Solver: the Hungarian method in its shortest-augmenting-path form
// (Munkres), started from the two-sided reduction (u_r = row minimum of M,
// v_c = column minimum of M - u) and a greedy matching on its zero reduced
// costs (see lap_start).  Each remaining free row is inserted by Dijkstra over
// columns with absolute tentative distances; the duals of the scanned tree are
// shifted once when an unmatched column is reached.  Ties are broken towards
// the lowest column index.
//
// Residual: the optimal dual is not unique, so the residual is taken under a
// canonical choice that does not depend on the solver's path:
//   column point: v^c = the greatest v <= 0 on the optimal dual face,
//                 u^c_r = min_q (M_rq - v^c_q);
//   row point:    u^r = the greatest u <= 0 on the optimal dual face,
//                 v^r_q = min_r (M_rq - u^r_r);
//   R = ((M - v^c - u^c) + (M - u^r - v^r)) / 2,
//   S = (sum u^c + sum v^c + sum u^r + sum v^r) / 2.
// With the solver's duals (u, v) and assignment sigma, v^c - v is the vector
// of shortest distances in the column graph whose arc c -> q costs the reduced
// cost M[sigma^-1(c)][q] - u - v >= 0, starting from label -v_q at every
// column: one dense Dijkstra pass.  The row point is the same on the row graph.
// With round-to-nearest arithmetic (FP64, or FP32 nearest) both residual
// halves are >= 0 exactly, because the subtracted dual is a row (column)
// minimum of the already rounded differences.  The FP32 certified variant is
// described at its code.
//
// What bounds it: the latency of a wave's serial chain (minimum over the lanes
// -> column -> its row -> next read of M) against the waves that a CU's LDS
// holds, then issue of vector instructions.  So the minimum runs on 32-bit keys
// (label_key), the solver's state stays in registers, LDS holds the matrix and
// two small tables, lane predicates are 64-bit wave masks on the scalar unit,
// and the start's matching works on the masks of comparisons.  Early blocks of
// N = 25 in FP64, two problems of n = 23 per wave: 3385 vector instructions a
// wave (4574 when the minimum ran on doubles and the start's matching read one
// column after the other), D -> C 815 -> 717 us (1.9 -> 2.1 TB/s of the block's
// read and write); certified FP32 574 -> 462 us; N = 31 FP64 3.32 -> 3.05 ms;
// N = 40 FP64 23.7 -> 21.0 ms.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

#include "lap_wave.hpp"
#include "rlt2_kernels.hpp"

namespace qap {

// Segment collectives for SEG in {4, 8, 16, 32, 64} lanes (all lanes of a
// segment active; segments independent).
template <int SEG>
struct SegS {
    static_assert(SEG == 4 || SEG == 8 || SEG == 16 || SEG == 32 || SEG == 64, "segment size");
    __device__ __forceinline__ static int lane() { return threadIdx.x & (SEG - 1); }

    template <typename T, typename Op>
    __device__ __forceinline__ static T reduce(T x, Op op) {
        x = op(x, dpp<kDppXor1>(x));
        x = op(x, dpp<kDppXor2>(x));
        if constexpr (SEG >= 8) x = op(x, dpp<kDppHalfMirror>(x));
        if constexpr (SEG >= 16) x = op(x, dpp<kDppMirror>(x));
        if constexpr (SEG >= 32) {
            T a, b;
            swap_pair<16>(x, a, b);
            x = op(a, b);
        }
        if constexpr (SEG >= 64) {
            T a, b;
            swap_pair<32>(x, a, b);
            x = op(a, b);
        }
        return x;
    }
    template <typename T>
    __device__ __forceinline__ static T min(T x) { return reduce(x, [](T a, T b) { return tmin(a, b); }); }
    // Sum of one value per lane, in one fixed order: pairs at stride 1, 2, 4,
    // ... bottom-up (addition being commutative, every lane gets the same bits).
    __device__ __forceinline__ static double sum(double x) { return reduce(x, [](double a, double b) { return a + b; }); }
    __device__ __forceinline__ static int imin(int x) {
        x = ::min(x, dpp_i<kDppXor1>(x));
        x = ::min(x, dpp_i<kDppXor2>(x));
        if constexpr (SEG >= 8) x = ::min(x, dpp_i<kDppHalfMirror>(x));
        if constexpr (SEG >= 16) x = ::min(x, dpp_i<kDppMirror>(x));
        if constexpr (SEG >= 32) {
            const unsigned u = (unsigned)x;
            auto r = __builtin_amdgcn_permlane16_swap(u, u, false, false);
            x = ::min((int)r[0], (int)r[1]);
        }
        if constexpr (SEG >= 64) {
            const unsigned u = (unsigned)x;
            auto r = __builtin_amdgcn_permlane32_swap(u, u, false, false);
            x = ::min((int)r[0], (int)r[1]);
        }
        return x;
    }
};

template <typename S>
__device__ __forceinline__ int seg_min(int x) { return S::imin(x); }
template <typename S>
__device__ __forceinline__ float seg_min(float x) { return S::min(x); }

// Wave masks seen as 64/SEG fields of SEG bits, one per segment.
template <int SEG>
struct SegBits {
    static constexpr unsigned long long kField = SEG == 64 ? ~0ull : (1ull << (SEG & 63)) - 1ull;
    // First lane of this lane's segment.
    __device__ __forceinline__ static int base() { return threadIdx.x & (64 - SEG); }
    // This lane's segment's bits of a wave mask (bit 0 = the segment's first lane).
    __device__ __forceinline__ static unsigned long long seg(unsigned long long b) {
        if constexpr (SEG == 64)
            return b;
        else
            return (b >> base()) & kField;
    }
    __device__ __forceinline__ static unsigned long long get(bool pred) { return seg(ballot64(pred)); }
    // Lowest set bit of every field.
    __device__ __forceinline__ static unsigned long long lowest(unsigned long long t) {
        if constexpr (SEG == 64) {
            return t & (0ull - t);
        } else if constexpr (SEG == 32) {
            const unsigned lo = (unsigned)t, hi = (unsigned)(t >> 32);
            return ((unsigned long long)(hi & (0u - hi)) << 32) | (lo & (0u - lo));
        } else {
            // -t in every field: ~t + 1 with the carry kept out of the next
            // field by adding without the fields' top bits.
            constexpr unsigned long long L = SEG == 16 ? 0x0001000100010001ull : 0x0101010101010101ull;
            constexpr unsigned long long H = L << (SEG - 1);
            const unsigned long long c = ~t;
            return t & (((c & ~H) + L) ^ (c & H));
        }
    }
};

// 32-bit keys of labels in an argmin.  Of a double the key is the high word,
// which keeps the order to 20 bits and so leaves almost always one candidate
// at the minimum, and a 32-bit minimum is one instruction per level where a
// double's is three (the cross-lane moves work on 32 bits).  The candidates'
// labels are then compared exactly ("settle" below); on the blocks of N = 25
// one below the first candidate's turns up in 1 to 5 of 100 passes.  Of a float
// the key is the label.  A lane that is out of the argmin gets the largest key.
//
// Distances (>= 0, up to the rounding of a tight arc): ordered as integers.
__device__ __forceinline__ int dist_key(double x, bool in) { return in ? __double2hiint(x) : 0x7fffffff; }
__device__ __forceinline__ float dist_key(float x, bool in) { return in ? x : __builtin_huge_valf(); }
// Labels of either sign: the high word read as a float, whose order it is for
// doubles below kBigLabel.
constexpr double kBigLabel = 0x1p1000;
__device__ __forceinline__ float label_key(double x, bool in)
{
    return in ? __int_as_float(__double2hiint(x)) : __builtin_huge_valf();
}
__device__ __forceinline__ float label_key(float x, bool in) { return in ? x : __builtin_huge_valf(); }

// x of lane j, j a scalar.
__device__ __forceinline__ float read_lane(float x, int j)
{
    return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(x), j));
}
__device__ __forceinline__ double read_lane(double x, int j)
{
    return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(x), j),
                            __builtin_amdgcn_readlane(__double2loint(x), j));
}

// x of lane `lane4 / 4` (any lane of the wave, given per lane).
__device__ __forceinline__ int from_lane(int lane4, int x) { return __builtin_amdgcn_ds_bpermute(lane4, x); }
__device__ __forceinline__ float from_lane(int lane4, float x)
{
    return __int_as_float(__builtin_amdgcn_ds_bpermute(lane4, __float_as_int(x)));
}
__device__ __forceinline__ double from_lane(int lane4, double x)
{
    return __hiloint2double(__builtin_amdgcn_ds_bpermute(lane4, __double2hiint(x)),
                            __builtin_amdgcn_ds_bpermute(lane4, __double2loint(x)));
}

// Per-problem LDS working set, for a problem of size n: the matrix (n rows of
// T, row stride n | 1), then n slots of scratch that each phase lays out for
// itself.  The odd row stride puts the rows a lane-per-row access reads (lane
// r reading row r) on distinct LDS banks; with an even n, lanes whose rows lie
// a multiple of 64 / gcd(n, 64) banks' worth apart would hit the same bank.
// The LDS a wave needs bounds how many waves a CU holds, and the kernels run
// faster the more it holds, so the scratch is what the largest phase takes: the
// two canonical passes' tables (a dual and an offset per node: 24 n bytes in
// FP64, 16 n in FP32), or the auction's prices, keys, owners and winners
// (24 n).  The hardware hands out LDS in steps of 1280 bytes: at n = 23 in FP64
// two problems take 9584 bytes, 8 steps, so that a CU holds 16 waves; with 48 n
// bytes of tables (9 steps, 14 waves) the same kernel was 10 % slower.
template <typename T, bool AUC = false>
struct LapLds {
    static constexpr int kSlot = AUC || sizeof(T) == 8 ? 24 : 16;   // scratch bytes per row
    __host__ __device__ static int row_stride(int n) { return n | 1; }
    __host__ __device__ static size_t mat_bytes(int n) {
        return (((size_t)n * row_stride(n) * sizeof(T)) + 15) & ~(size_t)15;
    }
    __host__ __device__ static size_t bytes(int n) { return mat_bytes(n) + (((size_t)n * kSlot + 15) & ~(size_t)15); }
};

template <typename T>
struct LapScratch {
    T* M;
    int ld;               // row stride of M (odd)
    unsigned char* tab;   // n * LapLds<T, AUC>::kSlot bytes
    __device__ LapScratch(unsigned char* base, int n)
        : M(reinterpret_cast<T*>(base)), ld(LapLds<T>::row_stride(n)), tab(base + LapLds<T>::mat_bytes(n)) {}
    // Array k of n values of type X.
    template <typename X>
    __device__ __forceinline__ X* arr(int n, int k) const { return reinterpret_cast<X*>(tab) + k * n; }
};

// LDS reads issued before any of them is used.
constexpr int kLapChunk = 8;

// f(r, x_r) for r = 0 .. n-1 with x_r = load(r): whole chunks of loads first,
// then the last partial one, whose indices past n - 1 re-read entry n - 1 and
// are not passed on unless `again` (f then sees entry n - 1 several times).
template <bool AGAIN, typename Load, typename F>
__device__ __forceinline__ void chunked(int n, Load load, F f)
{
    int r0 = 0;
    for (; r0 + kLapChunk <= n; r0 += kLapChunk) {
        decltype(load(0)) x[kLapChunk];
#pragma unroll
        for (int e = 0; e < kLapChunk; ++e) x[e] = load(r0 + e);
#pragma unroll
        for (int e = 0; e < kLapChunk; ++e) f(r0 + e, x[e]);
    }
    if (r0 < n) {
        decltype(load(0)) x[kLapChunk];
#pragma unroll
        for (int e = 0; e < kLapChunk; ++e) x[e] = load(min(r0 + e, n - 1));
#pragma unroll
        for (int e = 0; e < kLapChunk; ++e)
            if (AGAIN || r0 + e < n) f(r0 + e, x[e]);
    }
}

// Largest n of the wave's problems; UNI: all have the same, n is a scalar.
template <int SEG, bool UNI>
__device__ __forceinline__ int wave_size(int n)
{
    if constexpr (UNI) return n;
    int nw = 0;
#pragma unroll
    for (int g = 0; g < 64 / SEG; ++g) nw = ::max(nw, __builtin_amdgcn_readlane(n, g * SEG));
    return nw;
}

// The rows of this lane's column in global memory: entry r is at(r).
// LaneRows: a pointer and a stride (in entries) per lane.  WaveRows: one base
// pointer and stride (in bytes) for the wave and a 32-bit offset per lane, so
// that a row's address is scalar work.
template <typename T>
struct LaneRows {
    T* p;   // this lane's column in row 0
    long long ld;
    __device__ __forceinline__ T& at(int r) const
    {
        return *reinterpret_cast<T*>(reinterpret_cast<char*>(p) +
                                     (size_t)(unsigned)__umul24((unsigned)r, (unsigned)ld * (unsigned)sizeof(T)));
    }
};
template <typename T>
struct WaveRows {
    char* base;
    unsigned ldb;   // bytes
    unsigned off;   // bytes
    __device__ __forceinline__ T& at(int r) const
    {
        return *reinterpret_cast<T*>(base + (size_t)((unsigned)r * ldb) + off);
    }
};

// From two dual points to the residual and S: vc (this lane's column's dual of
// the column point), ur (its row's dual of the row point) and sg (its row's
// column, for `assign`).  The other halves of the two points are completed
// here: u^c_r = min_q (M_rq - v^c_q), v^r_q = min_r (M_rq - u^r_r).
// DOWN selects the FP32 certified completion (every written value rounded
// toward -inf); otherwise the completion runs in T with round-to-nearest and
// S is summed in FP64.
template <typename T, int SEG, bool DOWN, typename Rows>
__device__ __forceinline__ double lap_complete(const LapScratch<T>& sc, int n, const Rows& rows, bool write,
                                               T* __restrict__ duals, int32_t* __restrict__ assign, T vc, T ur, int sg)
{
    using S = SegS<SEG>;
    const T* __restrict__ M = sc.M;
    const int ldm = sc.ld;   // row stride of M
    const int l = S::lane();
    const bool ok = l < n;
    const T* __restrict__ Mrow = M + __umul24(ok ? l : 0, ldm);
    const T* __restrict__ Mcol = M + (ok ? l : 0);
    wave_sync();

    if constexpr (!DOWN) {
        // ---- round to nearest: residual = mean of the residuals under the
        // two points ----
        T* __restrict__ avc = sc.template arr<T>(n, 0);
        T* __restrict__ aur = sc.template arr<T>(n, 1);
        T* __restrict__ auc = sc.template arr<T>(n, 2);
        struct RowIn {
            T m, u, w;
        };
        if (ok) {
            avc[l] = vc;
            aur[l] = ur;
        }
        wave_sync();
        T uc = inf_of<T>(), vr = inf_of<T>();   // uc: lane as row; vr: lane as column
        if (ok) {
            chunked<true>(n, [&](int q) { return Mrow[q] - avc[q]; }, [&](int, T x) { uc = tmin(x, uc); });
            auc[l] = uc;
            chunked<true>(n, [&](int r) { return Mcol[__umul24(r, ldm)] - aur[r]; }, [&](int, T x) { vr = tmin(x, vr); });
        }
        wave_sync();
        if (ok && write) {
            chunked<false>(
                n, [&](int r) { return RowIn{Mcol[__umul24(r, ldm)], auc[r], aur[r]}; },
                [&](int r, const RowIn& x) { rows.at(r) = (T)0.5 * (((x.m - vc) - x.u) + ((x.m - x.w) - vr)); });
        }
        if (ok) {
            if (duals != nullptr) {
                duals[l] = uc;
                duals[n + l] = vc;
                duals[2 * n + l] = ur;
                duals[3 * n + l] = vr;
            }
            if (assign != nullptr) assign[l] = sg;
        }
        const double s = ok ? ((double)uc + (double)vc) + ((double)ur + (double)vr) : 0.0;
        wave_sync();
        return 0.5 * S::sum(s);
    } else {
        // ---- FP32 certified: the duals are completed in FP64 so that they
        // stay feasible (u_r + v_q <= M_rq exactly).  With U = (uc + ur)/2
        // and V = (vc + vr)/2 the residual M - U - V (the same value as the
        // mean of the two residuals) is then >= 0, and each entry and
        // S = sum U + sum V are written rounded down.
        //
        // A completed dual is a minimum of differences t = M - d.  Each
        // difference is computed once in round-to-nearest FP64, within
        // 2^-53 |t| of the exact one; as t - 2^-53 |t| increases with t, the
        // minimum m of the computed differences lowered by 2^-50 |m| (the
        // lowering itself rounding by at most 2^-53 of the result) lies below
        // every exact difference.  A residual entry M - V - U is computed in
        // two round-to-nearest steps, within 2.01 * 2^-53 (|M| + |V| + |U|)
        // of the exact value; lowered by 2^-50 times that sum (the lowering's
        // own rounding included), then by the float conversion toward -inf,
        // and clamped at 0 (the exact residual is >= 0), it is a valid lower
        // value.  Both replace per-operation directed rounding (TwoSum) with
        // a margin far below one FP32 step.
        double* __restrict__ au = sc.template arr<double>(n, 0);
        double* __restrict__ av = sc.template arr<double>(n, 1);
        if (ok) {
            au[l] = (double)vc;
            av[l] = (double)ur;
        }
        wave_sync();
        double uc = 0.0, vr = 0.0, U = 0.0, V = 0.0;
        if (ok) {
            uc = __builtin_huge_val();
            vr = __builtin_huge_val();
            chunked<true>(n, [&](int q) { return (double)Mrow[q] - au[q]; },
                          [&](int, double x) { uc = __builtin_fmin(uc, x); });
            chunked<true>(n, [&](int r) { return (double)Mcol[__umul24(r, ldm)] - av[r]; },
                          [&](int, double x) { vr = __builtin_fmin(vr, x); });
            uc -= __builtin_fabs(uc) * 0x1p-50;
            vr -= __builtin_fabs(vr) * 0x1p-50;
            U = 0.5 * add_down(uc, (double)ur);   // lane as row
            V = 0.5 * add_down((double)vc, vr);   // lane as column
        }
        wave_sync();
        if (ok) au[l] = U;
        wave_sync();
        if (ok && write) {
            const double aV = __builtin_fabs(V) * 0x1p-50;
            struct RowIn {
                T m;
                double u;
            };
            chunked<false>(
                n, [&](int r) { return RowIn{Mcol[__umul24(r, ldm)], au[r]}; },
                [&](int r, const RowIn& x) {
                    const double m = (double)x.m;
                    const double t = (m - V) - x.u;
                    // 2^-50 (|M| + |U| + |V|), the sum rounded once before
                    // the FMA and once in it: >= (1 - 2^-52) of the exact one.
                    const double margin = __builtin_fma(__builtin_fabs(m) + __builtin_fabs(x.u), 0x1p-50, aV);
                    rows.at(r) = to_float_down_nonneg(__builtin_fmax(t - margin, 0.0));
                });
        }
        if (ok) {
            if (duals != nullptr) {
                duals[l] = (T)uc;
                duals[n + l] = vc;
                duals[2 * n + l] = ur;
                duals[3 * n + l] = (T)vr;
            }
            if (assign != nullptr) assign[l] = sg;
        }
        // S = sum U + sum V rounded down: the sum of the lanes' U + V is taken
        // in round-to-nearest (one addition and at most six levels of pairwise
        // additions, so within (1 + 2^-53)^7 - 1 < 8 * 2^-53 of the exact sum
        // relative to the sum of magnitudes) and lowered by 2^-48 times the
        // round-to-nearest sum of the magnitudes, which covers that error and
        // the lowering's own rounding.
        const double s = S::sum(U + V), a = S::sum(__builtin_fabs(U) + __builtin_fabs(V));
        wave_sync();
        return s - a * 0x1p-48;
    }
}

// Start of the solver.  Row minima u_r of M, then column minima v_c of the
// reduced rows M_rc - u_r (the two-sided reduction: every reduced cost is
// >= 0 and each row and column has a zero), then a matching on the zeros:
// the rows in index order each take the lowest still free column c with
// M_rc - u_r = v_c.  On the structured blocks of the dual ascent this leaves
// far fewer rows free than a column reduction alone, and every free row costs
// Dijkstra steps.  A row's zeros are the wave mask of one comparison, so the
// matching runs on the scalar unit for all the wave's problems at once.
// On return aru[r] = u_r for every row r < n (kept through the Hungarian phase:
// a free row enters with that dual), v and prow (matched row or -1) for this
// lane's column; the result is the wave mask of the free rows (lane as row).
template <typename T, int SEG, bool UNI>
__device__ __forceinline__ unsigned long long lap_start(const LapScratch<T>& sc, int n, T* __restrict__ aru, T& v,
                                                        int& prow)
{
    const T* __restrict__ M = sc.M;
    const int ldm = sc.ld;   // row stride of M
    const int l = threadIdx.x & (SEG - 1);
    const bool ok = l < n;
    int* __restrict__ taken = sc.template arr<int>(n, sizeof(T) == 8 ? 2 : 1);   // after aru
    if (ok) {
        const T* __restrict__ Mr = M + __umul24(l, ldm);
        T um = Mr[0];
        chunked<true>(n, [&](int q) { return Mr[q]; }, [&](int, T x) { um = tmin(x, um); });
        aru[l] = um;
        taken[l] = -1;
    }
    wave_sync();
    const T* __restrict__ Mc = M + (ok ? l : 0);
    auto reduced = [&](int r) { return Mc[__umul24(r, ldm)] - aru[r]; };
    T vm = reduced(0);
    chunked<true>(n, reduced, [&](int, T x) { vm = tmin(x, vm); });
    v = vm;
    // The rows in order, counting for every column the rows that left it
    // free: the count stops at the row that takes it.  Rows past a problem's
    // n take no column.
    const int nw = wave_size<SEG, UNI>(n);
    const int last = ::max(n - 1, 0);
    unsigned long long freec = ballot64(ok);
    int cnt = 0;
    auto take = [&](unsigned long long z) __attribute__((always_inline)) {
        freec &= ~SegBits<SEG>::lowest(z & freec);
        cnt += lane_bit(freec) ? 1 : 0;
    };
    int r0 = 0;
    if constexpr (UNI) {   // whole chunks: no clamps, no rows past the end
        for (; r0 + kLapChunk <= n; r0 += kLapChunk) {
            T x[kLapChunk];
#pragma unroll
            for (int e = 0; e < kLapChunk; ++e) x[e] = reduced(r0 + e);
#pragma unroll
            for (int e = 0; e < kLapChunk; ++e) take(ballot64(x[e] == v));
        }
    }
    for (; r0 < nw; r0 += kLapChunk) {
        T x[kLapChunk];
#pragma unroll
        for (int e = 0; e < kLapChunk; ++e) x[e] = reduced(min(r0 + e, last));
#pragma unroll
        for (int e = 0; e < kLapChunk; ++e) take(ballot64(x[e] == v) & ballot64(r0 + e < n));
    }
    prow = ok && !lane_bit(freec) ? cnt : -1;
    if (prow >= 0) taken[prow] = l;
    wave_sync();
    return ballot64(ok && taken[ok ? l : 0] < 0);
}

// The two canonical passes side by side: the first SEG/2 lanes of a segment
// run the column pass and the other SEG/2 the row pass, each lane holding
// nodes h and h + SEG/2, so both take n steps together.  A relaxation is
// written (M - per-step dual) - per-node dual for both passes, and a step is
// branch-free but for near ties: it lowers every node's label, also the fixed
// ones' (whose labels can only change by the rounding of a tight arc), and a
// fixed node is masked out of the minimum.  The lowest node at
// the minimum is the minimum over the lanes of their lowest candidate's table
// offset, so no index arithmetic stands between the minimum and the table
// read.  On return (lane as column / as row) vc is the column-canonical dual
// of the lane's column, ur the row-canonical dual of its row and sg its row's
// column.  v, ucol, prow: this lane's column's dual, its matched row's dual and
// that row.
template <typename T, int SEG, bool UNI>
__device__ __forceinline__ void canonical_split(const LapScratch<T>& sc, int n, T v, T ucol, int prow, T& vc, T& ur,
                                                int& sg)
{
    constexpr int H = SEG / 2;
    using HS = SegS<H>;
    const int l = threadIdx.x & (SEG - 1);
    const bool ok = l < n;
    // Tables of the column pass (node = column) and the row pass (node = row):
    // the dual subtracted first when node f is fixed, and the byte offset its
    // key adds to a node's place in M.
    T* __restrict__ sc_c = sc.template arr<T>(n, 0);
    T* __restrict__ sc_r = sc_c + n;
    int* __restrict__ off_c = sc.template arr<int>(n, 2 * (int)(sizeof(T) / sizeof(int)));   // after both
    int* __restrict__ off_r = off_c + n;
    const int rowb = sc.ld * (int)sizeof(T);
    wave_sync();
    if (ok || (n == 0 && l == 0)) {
        // A column without a row (non-finite costs) stands for offset 0, and
        // so does a row without a column; an empty problem has one entry.
        sc_c[l] = ucol;
        off_c[l] = (int)__umul24(prow < 0 ? 0 : prow, rowb);
        sc_r[l] = v;
        off_r[l] = 0;
    }
    wave_sync();
    if (ok && prow >= 0) {
        sc_r[prow] = v;
        off_r[prow] = l * (int)sizeof(T);
    }
    wave_sync();
    const bool rowpass = l >= H;
    const int h = l & (H - 1);
    // A node is 4 times its number: the offset of its entry in an int array and,
    // modulo 4 H, of its lane in the half segment.
    const char* const tab_s = reinterpret_cast<const char*>(rowpass ? sc_r : sc_c);
    const char* const tab_o = reinterpret_cast<const char*>(rowpass ? off_r : off_c);
    const int last = ::max(n - 1, 0) * 4;
    const int half4 = (int)(threadIdx.x & (64 - H)) * 4;   // 4 x the half segment's first lane
    const char* const m0 = reinterpret_cast<const char*>(sc.M);
    int node[2];         // an absent node repeats node 0
    const char* mq[2];
    T lab[2], w[2];
    unsigned long long fxm[2];   // fixed (or absent) node, as wave masks
    for (int q = 0; q < 2; ++q) {
        const int t = h + q * H;
        const int tc = t < n ? t : 0;
        node[q] = tc * 4;
        mq[q] = m0 + (rowpass ? (int)__umul24(tc, rowb) : tc * (int)sizeof(T));
        fxm[q] = ballot64(t >= n);
        // The node's own dual: v of a column; of a row, what its column's
        // entry holds.
        const T vq = from_lane((SegBits<SEG>::base() + tc) * 4, v);
        const T uq = sc_c[(unsigned)off_r[tc] / (unsigned)sizeof(T)];
        w[q] = rowpass ? uq : vq;
        lab[q] = -w[q];
    }
    // Every segment takes the wave's largest n steps, so the loop counter is
    // scalar: a segment past its own n has every node fixed, and its further
    // steps relax from an infinite label.
    const int nw = wave_size<SEG, UNI>(n);
    // Labels stay between the smallest and the largest start label.
    const bool big = sizeof(T) == 8 && (ballot64(__builtin_fabs((double)w[0]) >= kBigLabel) |
                                        ballot64(__builtin_fabs((double)w[1]) >= kBigLabel)) != 0ull;
    for (int step = 0; step < nw; ++step) {
        const float k0 = label_key(lab[0], !lane_bit(fxm[0])), k1 = label_key(lab[1], !lane_bit(fxm[1]));
        const float kmin = HS::min(tmin(k0, k1));
        unsigned long long e0 = ballot64(k0 == kmin) & ~fxm[0], e1 = ballot64(k1 == kmin) & ~fxm[1];
        if (__builtin_expect(big, 0)) {   // every node left is a candidate
            e0 = ~fxm[0];
            e1 = ~fxm[1];
        }
        int f = lane_bit(e1) ? node[1] : last;
        f = HS::imin(lane_bit(e0) ? node[0] : f);
        T dmin = kmin;
        unsigned long long is1 = ballot64(node[1] == f);
        T s = *reinterpret_cast<const T*>(tab_s + f * (int)(sizeof(T) / sizeof(int)));
        int off = *reinterpret_cast<const int*>(tab_o + f);
        if constexpr (sizeof(T) == 8) {
            // The label of node f, from its lane.
            auto label = [&]() __attribute__((always_inline)) {
                return from_lane((f & (4 * (H - 1))) | half4, lane_bit(is1) ? lab[1] : lab[0]);
            };
            dmin = label();
            // Settle: while some candidate's label is below the chosen one's,
            // choose among those.
            unsigned long long b0 = ballot64(lab[0] < dmin) & e0, b1 = ballot64(lab[1] < dmin) & e1;
            if (__builtin_expect((b0 | b1) != 0ull, 0)) {
                do {
                    int g = lane_bit(b1) ? node[1] : INT32_MAX;
                    g = HS::imin(lane_bit(b0) ? node[0] : g);
                    f = g != INT32_MAX ? g : f;
                    is1 = ballot64(node[1] == f);
                    dmin = label();
                    b0 &= ballot64(lab[0] < dmin);
                    b1 &= ballot64(lab[1] < dmin);
                } while ((b0 | b1) != 0ull);
                s = *reinterpret_cast<const T*>(tab_s + f * (int)(sizeof(T) / sizeof(int)));
                off = *reinterpret_cast<const int*>(tab_o + f);
            }
            if (!UNI) dmin = step < n ? dmin : inf_of<T>();
        }
        fxm[0] |= ballot64(node[0] == f);
        fxm[1] |= is1;
        for (int q = 0; q < 2; ++q) {
            const T m = *reinterpret_cast<const T*>(mq[q] + off);
            lab[q] = tmin(lab[q], dmin + ((m - s) - w[q]));
        }
    }
    wave_sync();
    // v^c = v + x by column, u^r = u + y by row.
    T* __restrict__ avc = sc.template arr<T>(n, 0);
    T* __restrict__ aur = sc.template arr<T>(n, 1);
    int* __restrict__ asg = reinterpret_cast<int*>(sc.template arr<T>(n, 2));
    for (int q = 0; q < 2; ++q) {
        const int t = h + q * H;
        if (t < n) (rowpass ? aur : avc)[t] = w[q] + lab[q];
    }
    if (ok && prow >= 0) asg[prow] = l;
    wave_sync();
    const int lc = ok ? l : 0;
    vc = n > 0 ? avc[lc] : T(0);
    ur = n > 0 ? aur[lc] : T(0);
    sg = n > 0 ? asg[lc] : 0;
}

// Solve, canonicalise and write residuals for the n x n matrix sc.M (in LDS,
// row stride sc.ld, left unchanged).  The residual goes to `rows` when
// `write`, duals (nullable) get [uc | vc | ur | vr], assign (nullable) the
// solver's assignment.  Returns S to every lane of the segment.  Called by
// whole waves; segments may have different n (0 <= n <= SEG), unless UNI (n is
// then a scalar).
//
// The free rows of all the wave's problems are inserted in one loop: each
// pass, every segment that still has a free row takes one Dijkstra step, and a
// segment whose step reached an unmatched column augments and starts on its
// next free row while the others go on, so a wave runs as many passes as its
// busiest problem needs rather than the sum over rows of the busiest problem
// per row.  The column reached is the lowest candidate of the key minimum.  An
// augmenting path is walked on the scalar unit, one segment at a time.  Every pass of an active segment
// adds a column to its tree or uses up a free row, so the loop ends.
template <typename T, int SEG, bool DOWN, bool UNI, typename Rows>
__device__ __forceinline__ double lap_concentrate(const LapScratch<T>& sc, int n, const Rows& rows, bool write,
                                                  T* __restrict__ duals, int32_t* __restrict__ assign)
{
    using S = SegS<SEG>;
    using Bits = SegBits<SEG>;
    constexpr int LPW = 64 / SEG;
    const int l = S::lane();
    const bool ok = l < n;
    const T INF = inf_of<T>();
    T* __restrict__ aru = sc.template arr<T>(n, 0);   // row minima: the dual a free row enters with
    const int rowb = sc.ld * (int)sizeof(T);
    const char* const Mcol = reinterpret_cast<const char*>(sc.M + (ok ? l : 0));

    T v;         // dual of this lane's column
    int prow;    // row matched to it, -1 when free
    unsigned long long freem = lap_start<T, SEG, UNI>(sc, n, aru, v, prow);   // free rows (lane as row)
    T ucol = prow >= 0 ? aru[prow] : (T)0;   // dual of the matched row

    // Lane predicates as wave masks: the columns in range, those already in
    // their problem's shortest-path tree, the lanes of problems still
    // inserting a row.
    const unsigned long long okm = ballot64(ok);
    unsigned long long usedm = 0, actm = 0;
    T dist = INF;          // tentative distance of this lane's column
    int way = -1;          // 4 x lane of the column it was reached through, -1: the new row
    int row = -1;          // row being inserted
    T urow = 0, ui0 = 0;   // its dual, and the dual of the row being scanned
    int i0b = 0;           // byte offset of the row being scanned
    T d0 = 0;              // distance at which that row was reached
    int j0 = -1;           // 4 x lane of the column through which it was reached
    // The next free row of the segment whose lanes are segm (first lane base).
    auto next_row = [&](unsigned long long segm, int base) __attribute__((always_inline)) {
        const unsigned long long f = freem & segm;
        freem &= ~(f & (0ull - f));
        const int r = f ? (int)__builtin_ctzll(f) - base : -1;
        actm = f ? (actm | segm) : (actm & ~segm);
        usedm &= ~segm;
        const int rc = ::max(r, 0);
        const T u0 = aru[rc];
        const int rb = (int)__umul24(rc, rowb);
        if (lane_bit(segm)) {
            row = r;
            urow = u0;
            ui0 = u0;
            i0b = rb;
            d0 = 0;
            j0 = -1;
            dist = INF;
            way = -1;
        }
    };
#pragma unroll
    for (int g = 0; g < LPW; ++g) next_row(Bits::kField << (g * SEG), g * SEG);

    const int base4 = Bits::base() * 4;
    while (actm != 0ull) {
        const unsigned long long livem = actm & okm & ~usedm;
        const T m = *reinterpret_cast<const T*>(Mcol + i0b);
        const T cur = d0 + ((m - ui0) - v);
        const bool better = lane_bit(ballot64(cur < dist) & livem);
        dist = better ? cur : dist;
        way = better ? j0 : way;
        const auto key = dist_key(dist, lane_bit(livem));
        const auto kmin = seg_min<S>(key);
        unsigned long long cand = ballot64(key == kmin) & livem;
        // The column reached (j4 = 4 x its lane), and what its lane holds: its
        // distance, its row and that row's dual.  Settle (FP64): while some
        // candidate's distance is below the chosen one's, choose among those.
        // Segments without a candidate (not active) read some lane; what they
        // read is not used.
        int j4, p;
        T dmin = (T)kmin;   // FP32: the distance itself
        if constexpr (LPW == 1) {
            // One problem: scalars throughout.
            int j = (int)__builtin_ctzll(cand);
            if constexpr (sizeof(T) == 8) {
                dmin = read_lane(dist, j);
                unsigned long long below = ballot64(dist < dmin) & cand;
                while (__builtin_expect(below != 0ull, 0)) {
                    j = (int)__builtin_ctzll(below);
                    dmin = read_lane(dist, j);
                    below &= ballot64(dist < dmin);
                }
            }
            p = __builtin_amdgcn_readlane(prow, j);
            ui0 = read_lane(ucol, j);
            j4 = j * 4;
            usedm |= 1ull << j;
        } else {
            auto lowest4 = [&](unsigned long long c) __attribute__((always_inline)) -> int {
                return base4 + (int)__builtin_ctz((unsigned)Bits::seg(c) | (SEG < 32 ? 1u << (SEG & 31) : 0u)) * 4;
            };
            j4 = lowest4(cand);
            if constexpr (sizeof(T) == 8) dmin = from_lane(j4, dist);
            p = from_lane(j4, prow);
            ui0 = from_lane(j4, ucol);
            if constexpr (sizeof(T) == 8) {
                unsigned long long below = ballot64(dist < dmin) & cand;
                if (__builtin_expect(below != 0ull, 0)) {
                    do {
                        const bool has = Bits::seg(below) != 0ull;
                        const int jb = lowest4(below);
                        j4 = has ? jb : j4;
                        dmin = from_lane(j4, dist);
                        below &= ballot64(dist < dmin);
                    } while (below != 0ull);
                    p = from_lane(j4, prow);
                    ui0 = from_lane(j4, ucol);
                }
            }
            usedm |= ballot64(j4 == base4 + 4 * l);
        }
        i0b = (int)__umul24(::max(p, 0), rowb);
        d0 = dmin;
        j0 = j4;
        // Segments whose column is unmatched.
        unsigned long long augm = LPW == 1 ? (p < 0 ? actm : 0ull) : actm & ballot64(p < 0);
        if (augm == 0ull) continue;
        do {
            const int base = (int)__builtin_ctzll(augm);
            const unsigned long long segm = Bits::kField << base;
            augm &= ~segm;
            // Dual shift of the scanned tree (the reached column has dist =
            // dmin, so its shift is 0).
            if (lane_bit(usedm & segm)) {
                const T sh = dmin - dist;
                v -= sh;
                ucol += sh;
            }
            // The path from the reached column back to the new row: a column
            // on it takes the row and row dual of its predecessor, the first
            // one the new row.
            unsigned long long onm = 0;
            int j = __builtin_amdgcn_readlane(j4, base) >> 2;
            for (int hop = 0; j >= 0 && hop < SEG; ++hop) {
                onm |= 1ull << j;
                j = __builtin_amdgcn_readlane(way, j) >> 2;
            }
            const int pw = from_lane(way, prow);
            const T uw = from_lane(way, ucol);
            if (lane_bit(onm)) {
                prow = way >= 0 ? pw : row;
                ucol = way >= 0 ? uw : urow + dmin;
            }
            next_row(segm, base);
        } while (augm != 0ull);
    }

    T vc, ur;
    int sg;
    canonical_split<T, SEG, UNI>(sc, n, v, ucol, prow, vc, ur, sg);
    return lap_complete<T, SEG, DOWN>(sc, n, rows, write, duals, assign, vc, ur, sg);
}

}  // namespace qap
