// Launch code of one precision mode: the kernels of one dual-ascent iteration
// (Algorithm 1 of arXiv 1510.02065), the certification cascade, the initial dual, the batched assignment solve and
// the children of a branch-and-bound node.  Included by ops_f64.hip,
// ops_f32d.hip and ops_f32n.hip, each of which instantiates Ops<PM> for one
// mode, so the three modes compile in parallel.
#pragma once
#include "handle.hpp"

namespace qap {

namespace {

template <int PM, int SEG, bool AUC>
hipError_t launch_family_seg(qap_rlt2* h, int famk, const ClassHost& c, double* values)
{
    using T = StoreT<PM>;
    constexpr int LPW = 64 / SEG;
    const size_t lds = slot_lds<T, SEG, AUC>(c.nmax);
    if (lds > h->lds_limit) return hipErrorInvalidConfiguration;   // not launched
    T* D = static_cast<T*>(h->dD);
    T* C = static_cast<T*>(h->dC);
    T* B = static_cast<T*>(h->dB);
    return in_launches((c.total + LPW - 1) / LPW, 64, [&](long long first, unsigned grid) {
        const FamilyClass fc = c.dev(first * LPW);
        if (famk == kFamD)
            hipLaunchKernelGGL((k_lap_family_s<PM, SEG, kFamD, AUC>), dim3(grid), dim3(64), lds, h->stream, D, C, B,
                               h->dInst, fc, c.nmax, values, h->dmode, h->dAct);
        else
            hipLaunchKernelGGL((k_lap_family_s<PM, SEG, kFamC, AUC>), dim3(grid), dim3(64), lds, h->stream, D, C, B,
                               h->dInst, fc, c.nmax, values, kAllBlocks, h->dAct);
        return hipGetLastError();
    });
}

template <int PM, int SEG, bool AUC>
hipError_t launch_B_seg(qap_rlt2* h, const ClassHost& c)
{
    using T = StoreT<PM>;
    constexpr int LPW = 64 / SEG;
    const size_t lds = slot_lds<T, SEG, AUC>(c.nmax);
    if (lds > h->lds_limit) return hipErrorInvalidConfiguration;
    const unsigned grid = (unsigned)((c.total + LPW - 1) / LPW);   // a wave per instance at most
    const bool tr = h->trace_level >= 1;
    hipLaunchKernelGGL((k_lap_B_s<PM, SEG, AUC>), dim3(grid), dim3(64), lds, h->stream, static_cast<T*>(h->dB),
                       h->dInst, c.dev(0), c.nmax, h->dLB, tr ? h->dTrace : nullptr, h->dCounter, kTraceRows, h->K,
                       h->trace_level >= 2 ? h->dValB : nullptr, h->dSigma, h->dAct, h->dStop);
    return hipGetLastError();
}

// Lanes per problem: the narrowest segment that holds the class's problems
// (seg_for), one column per lane.  Several columns per lane put more problems
// in a wave, but the wave runs as many Dijkstra passes as its busiest problem
// needs and holds more LDS, so a CU holds fewer waves: at n = 23 in FP64,
// 0.97 ms for 32 lanes x 1 column, 1.29 for 16 x 2 and 2.46 for 8 x 3; at
// n = 38, 27 ms for 64 x 1 and 41 for 32 x 2.
#define QAP_BY_SEG(SEGV, CALL)   \
    switch (SEGV) {              \
    case 8: return CALL(8);      \
    case 16: return CALL(16);    \
    case 32: return CALL(32);    \
    default: return CALL(64);    \
    }

template <int PM>
hipError_t launch_family_class(qap_rlt2* h, int famk, const ClassHost& c, double* values)
{
    if (c.total <= 0) return hipSuccess;
    if (h->lap_solver == QAP_LAP_SOLVER_AUCTION) {
#define QAP_CALL(SG) launch_family_seg<PM, SG, true>(h, famk, c, values)
        QAP_BY_SEG(c.seg, QAP_CALL)
#undef QAP_CALL
    }
#define QAP_CALL(SG) launch_family_seg<PM, SG, false>(h, famk, c, values)
    QAP_BY_SEG(c.seg, QAP_CALL)
#undef QAP_CALL
}

template <int PM>
hipError_t launch_family(qap_rlt2* h, int famk, double* values)
{
    for (const ClassHost& c : h->fam[famk]) {
        hipError_t e = launch_family_class<PM>(h, famk, c, values);
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

template <int PM>
hipError_t launch_B_class(qap_rlt2* h, const ClassHost& c)
{
    if (c.total <= 0) return hipSuccess;
    if (h->lap_solver == QAP_LAP_SOLVER_AUCTION) {
#define QAP_CALL(SG) launch_B_seg<PM, SG, true>(h, c)
        QAP_BY_SEG(c.seg, QAP_CALL)
#undef QAP_CALL
    }
#define QAP_CALL(SG) launch_B_seg<PM, SG, false>(h, c)
    QAP_BY_SEG(c.seg, QAP_CALL)
#undef QAP_CALL
}

template <int PM>
hipError_t launch_B(qap_rlt2* h)
{
    for (const ClassHost& c : h->fam[2]) {
        hipError_t e = launch_B_class<PM>(h, c);
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

template <int PM, int SEG, bool AUC>
hipError_t launch_batch_seg(hipStream_t st, int nmax, int count, const int* range, const int32_t* idx,
                            const int32_t* n, const int64_t* mo, const int64_t* vo, StoreT<PM>* cost, double* value,
                            StoreT<PM>* duals, int32_t* assign, int wr)
{
    using T = StoreT<PM>;
    if (count <= 0) return hipSuccess;
    constexpr int LPW = 64 / SEG;
    const size_t lds = slot_lds<T, SEG, AUC>(nmax);
    return in_launches(((long long)count + LPW - 1) / LPW, 64, [&](long long first, unsigned grid) {
        hipLaunchKernelGGL((k_lap_batch<PM, SEG, AUC>), dim3(grid), dim3(64), lds, st, first, count, range, idx, nmax,
                           n, mo, vo, cost, value, duals, assign, wr);
        return hipGetLastError();
    });
}

// Workgroups of k_sweep_triple<PM, NT> a CU holds at size N (its registers
// and its LDS); 0 when the triple does not fit NT threads.
template <int PM, int NT>
int triple_per_cu(int N)
{
    const size_t lds = sweep_triple_lds<StoreT<PM>, NT>(N);
    if (lds == (size_t)-1) return 0;
    int nb = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, k_sweep_triple<PM, NT>, NT, lds) != hipSuccess) {
        (void)hipGetLastError();
        return 0;
    }
    return nb;
}

template <int PM, int BS>
hipError_t launch_box(qap_rlt2* h, const SweepClass& c)
{
    using T = StoreT<PM>;
    using Shape = BoxShape<BS>;
    constexpr size_t lds = Shape::template lds<T>();
    if (lds > h->lds_limit) return hipErrorInvalidConfiguration;
    hipLaunchKernelGGL((k_sweep_box<PM, BS>), dim3((unsigned)c.nwg), dim3(Shape::NT), lds, h->stream,
                       static_cast<T*>(h->dD), static_cast<const T*>(h->dCC), static_cast<T*>(h->dB), h->dTri, h->dInst,
                       c.d_pre, c.d_ids, (int)c.ids.size(), h->dAct);
    return hipGetLastError();
}

// Steps 1-3 over the instances of one size.  kSweepBox: one workgroup per
// (j, n) tile pair of a triple.  Otherwise everything of a triple goes
// through LDS: when a CU holds only one triple's workgroup, one persistent
// workgroup per CU walks the triples and overlaps each triple's start with the
// previous one's tiles; when it holds two or more (nt > 0), one workgroup of
// nt threads per triple lets the hardware overlap them.  The workgroup that
// takes an instance's first triple clears its B.
template <int PM>
hipError_t launch_sweep(qap_rlt2* h, const SweepClass& c)
{
    using T = StoreT<PM>;
    T* B = static_cast<T*>(h->dB);
    T* D = static_cast<T*>(h->dD);
    const T* CC = static_cast<const T*>(h->dCC);
    const int K = (int)c.ids.size();
    if (c.nt == kSweepBox) {
        switch (box_edge<T>(c.N)) {
#define QAP_BOX(BS) \
    case BS: return launch_box<PM, BS>(h, c);
            QAP_BOX(15) QAP_BOX(16)
            default:
                if constexpr (PM == kPrecF64) {
                    switch (box_edge<T>(c.N)) { QAP_BOX(11) QAP_BOX(12) QAP_BOX(13) QAP_BOX(14) }
                } else {
                    switch (box_edge<T>(c.N)) {
                        QAP_BOX(17) QAP_BOX(18) QAP_BOX(19) QAP_BOX(20) QAP_BOX(21) QAP_BOX(22)
                    }
                }
#undef QAP_BOX
        }
        return hipErrorInvalidConfiguration;
    }
    if (c.nt == kTripleThreadsSmall) {
        const size_t lds = sweep_triple_lds<T, kTripleThreadsSmall>(c.N);
        if (lds == (size_t)-1) return hipErrorInvalidConfiguration;
        hipLaunchKernelGGL((k_sweep_triple<PM, kTripleThreadsSmall>), dim3((unsigned)c.nwg), dim3(kTripleThreadsSmall),
                           lds, h->stream, D, CC, B, h->dTri, h->dInst, c.d_pre, c.d_ids, K, h->dAct);
    } else if (c.nt == kTripleThreads) {
        const size_t lds = sweep_triple_lds<T>(c.N);
        hipLaunchKernelGGL((k_sweep_triple<PM, kTripleThreads>), dim3((unsigned)c.nwg), dim3(kTripleThreads), lds,
                           h->stream, D, CC, B, h->dTri, h->dInst, c.d_pre, c.d_ids, K, h->dAct);
    } else {
        const size_t lds = sweep_triple_lds<T>(c.N);
        const long long grid = std::min<long long>(c.nwg, h->num_cu);
        hipLaunchKernelGGL((k_sweep_triple_p<PM>), dim3((unsigned)grid), dim3(kTripleThreads), lds, h->stream, D, CC,
                           B, h->dTri, h->dInst, c.d_pre, c.d_ids, K, c.nwg, c.N, h->dAct);
    }
    return hipGetLastError();
}

}  // namespace

template <int PM>
int Ops<PM>::sweep_threads(int N, size_t lds_limit)
{
    using T = StoreT<PM>;
    if (sweep_triple_lds<T>(N) > lds_limit) return kSweepBox;
    // The smaller workgroup when a CU holds two or more of them, else the larger
    // one when a CU holds two or more, else 0 (persistent).  Smaller
    // workgroups keep more triples in flight per CU, each waiting at its own
    // barriers: on the 256-node batch in certified FP32 the 512-thread sweeps
    // took 5.7 ms per iteration where the 1024-thread ones, holding more
    // waves, took 8.7 ms.
    if (triple_per_cu<PM, kTripleThreadsSmall>(N) >= 2) return kTripleThreadsSmall;
    if (triple_per_cu<PM, kTripleThreads>(N) >= 2) return kTripleThreads;
    return 0;
}

template <int PM>
int Ops<PM>::sweep_tiles(int N)
{
    return box_tiles<StoreT<PM>>(N);
}

template <int PM, bool SPREAD>
hipError_t launch_transfer_C(qap_rlt2* h)
{
    using T = StoreT<PM>;
    return in_launches(h->totalP, 256, [&](long long first, unsigned grid) {
        hipLaunchKernelGGL((k_transfer_C<PM, SPREAD>), dim3(grid), dim3(256), 0, h->stream, static_cast<T*>(h->dC),
                           static_cast<const T*>(h->dB), h->dInst, h->dPreP, h->K, first, h->dAct);
        return hipGetLastError();
    });
}

template <int PM>
hipError_t launch_clear_B(qap_rlt2* h)
{
    return in_launches(groups_of(h->totalB, 256), 256, [&](long long first, unsigned grid) {
        hipLaunchKernelGGL((k_clear_B<PM>), dim3(grid), dim3(256), 0, h->stream, static_cast<StoreT<PM>*>(h->dB),
                           h->dPreB, h->K, h->totalB, first * 256, h->dAct);
        return hipGetLastError();
    });
}

template <int PM>
hipError_t launch_spread_prep(qap_rlt2* h)
{
    using T = StoreT<PM>;
    return in_launches(groups_of(h->totalC, 256), 256, [&](long long first, unsigned grid) {
        hipLaunchKernelGGL((k_spread_prep<PM>), dim3(grid), dim3(256), 0, h->stream, static_cast<T*>(h->dC),
                           static_cast<T*>(h->dB), static_cast<T*>(h->dCC), h->dInst, h->dPreC, h->K, h->totalC,
                           first * 256, h->dAct);
        return hipGetLastError();
    });
}

// Steps 1 and 5 of a level-1 iteration in one pass over C.
template <int PM>
hipError_t Ops<PM>::enqueue_spread_transfer(qap_rlt2* h)
{
    const hipError_t e = launch_transfer_C<PM, true>(h);
    return e == hipSuccess ? launch_clear_B<PM>(h) : e;
}

template <int PM>
hipError_t Ops<PM>::enqueue_step(qap_rlt2* h, int step)
{
    using T = StoreT<PM>;
    T* B = static_cast<T*>(h->dB);
    T* C = static_cast<T*>(h->dC);
    T* D = static_cast<T*>(h->dD);
    T* CC = static_cast<T*>(h->dCC);
    hipStream_t st = h->stream;
    const bool vals = h->trace_level >= 2;
    switch (step) {
    case 3: {   // steps 1-3 (level 1: step 1)
        if (h->level == 1) {
            const hipError_t e = in_launches(groups_of(h->totalC, 256), 256, [&](long long first, unsigned grid) {
                hipLaunchKernelGGL((k_spread_B<PM>), dim3(grid), dim3(256), 0, st, C, B, h->dInst, h->dPreC, h->K,
                                   h->totalC, first * 256, h->dAct);
                return hipGetLastError();
            });
            return e == hipSuccess ? launch_clear_B<PM>(h) : e;
        }
        hipError_t e = launch_spread_prep<PM>(h);
        if (e != hipSuccess) return e;
        if (h->dmode == kAllBlocks)
            return in_launches(h->totalWG, 256, [&](long long first, unsigned grid) {
                hipLaunchKernelGGL((k_sweep<PM>), dim3(grid), dim3(256), 0, st, D, CC, B, h->dTri, h->dInst,
                                   h->dPreWG, h->K, first, h->dAct);
                return hipGetLastError();
            });
        for (const SweepClass& c : h->sweep_cls) {
            e = launch_sweep<PM>(h, c);
            if (e != hipSuccess) return e;
        }
        return hipSuccess;
    }
    case 4:
        if (h->level == 1) return hipSuccess;
        return launch_family<PM>(h, kFamD, vals ? h->dValD : nullptr);
    case 5:
        return launch_transfer_C<PM, false>(h);
    case 6:
        return launch_family<PM>(h, kFamC, vals ? h->dValC : nullptr);
    case 7:
        return launch_B<PM>(h);
    default:
        return hipErrorInvalidValue;
    }
}

template <int PM>
hipError_t Ops<PM>::enqueue_sweep_concentrate_overlapped(qap_rlt2* h)
{
    hipStream_t A = h->stream, Bs = h->stream2;
    hipError_t e = launch_spread_prep<PM>(h);
    if (e != hipSuccess) return e;
    if ((e = hipEventRecord(h->ev_fork, A)) != hipSuccess) return e;
    if ((e = hipStreamWaitEvent(Bs, h->ev_fork, 0)) != hipSuccess) return e;
    for (size_t i = 0; i < h->sweep_cls.size() && e == hipSuccess; ++i) {
        const SweepClass& c = h->sweep_cls[i];
        e = launch_sweep<PM>(h, c);
        if (e == hipSuccess) e = hipEventRecord(h->ev_size[i], A);
        if (e == hipSuccess) e = hipStreamWaitEvent(Bs, h->ev_size[i], 0);
        if (e != hipSuccess) break;
        // The concentration of this size, on the second stream.
        h->stream = Bs;
        e = launch_family_class<PM>(h, kFamD, h->famD_size[i], h->trace_level >= 2 ? h->dValD : nullptr);
        h->stream = A;
    }
    if (e != hipSuccess) return e;
    if ((e = hipEventRecord(h->ev_join, Bs)) != hipSuccess) return e;
    return hipStreamWaitEvent(A, h->ev_join, 0);
}

template <int PM>
hipError_t Ops<PM>::certify(qap_rlt2* h)
{
    using T = StoreT<PM>;
    hipStream_t st = h->stream;
    const T *D = static_cast<const T*>(h->dD), *C = static_cast<const T*>(h->dC), *B = static_cast<const T*>(h->dB);
    hipError_t e = hipSuccess;
    if (h->level == 1)
        e = in_launches(groups_of(h->totalC, 256), 256, [&](long long first, unsigned grid) {
            hipLaunchKernelGGL((k_cert_noD<T>), dim3(grid), dim3(256), 0, st, C, h->dCt, h->totalC, first);
            return hipGetLastError();
        });
    else if (h->dmode == kAllBlocks)
        e = in_launches(groups_of(h->totalC, 4), 256, [&](long long first, unsigned grid) {
            hipLaunchKernelGGL((k_cert_D<T>), dim3(grid), dim3(256), 0, st, D, C, h->dCt, h->dInst, h->dPreC, h->K,
                               h->totalC, first);
            return hipGetLastError();
        });
    else
        e = in_launches(h->totalCert, kCertThreads, [&](long long first, unsigned grid) {
            hipLaunchKernelGGL((k_cert_pairs<T>), dim3(grid), dim3(kCertThreads), 0, st, D, C, h->dCt, h->dInst,
                               h->dPreCert, h->K, first);
            return hipGetLastError();
        });
    if (e != hipSuccess) return e;
    e = in_launches(groups_of(h->totalB, 4), 256, [&](long long first, unsigned grid) {
        hipLaunchKernelGGL((k_cert_C<T>), dim3(grid), dim3(256), 0, st, h->dCt, B, h->dBt, h->dInst, h->dPreB, h->K,
                           h->totalB, first);
        return hipGetLastError();
    });
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_cert_final<>, dim3(h->K), dim3(64), 0, st, h->dBt, h->dLB, h->dCert, h->dInst);
    return hipGetLastError();
}

template <int PM>
hipError_t Ops<PM>::init_instance(qap_rlt2* h, int k, const double* dF, const double* dDm, const double* dB0)
{
    using T = StoreT<PM>;
    const Inst& I = h->inst[k];
    const int N = I.N;
    const long long nC = (long long)N * N * (N - 1) * (N - 1);
    hipLaunchKernelGGL((k_init<PM>), dim3((unsigned)groups_of(nC, 256)), dim3(256), 0, h->stream, dF, dDm, dB0,
                       static_cast<T*>(h->dB) + I.offB, static_cast<T*>(h->dC) + I.offC, N);
    return hipGetLastError();
}

template <int PM>
hipError_t Ops<PM>::lap_batch(hipStream_t st, int nmax, int count, const int* range, const int32_t* idx,
                              const int32_t* n, const int64_t* mo, const int64_t* vo, void* cost, double* value,
                              void* duals, int32_t* assign, int wr, int solver)
{
    using T = StoreT<PM>;
    T* c = static_cast<T*>(cost);
    T* d = static_cast<T*>(duals);
#define QAP_SEG(SG)                                                                                            \
    return solver == QAP_LAP_SOLVER_AUCTION                                                                    \
               ? launch_batch_seg<PM, SG, true>(st, nmax, count, range, idx, n, mo, vo, c, value, d, assign, wr)  \
               : launch_batch_seg<PM, SG, false>(st, nmax, count, range, idx, n, mo, vo, c, value, d, assign, wr)
    switch (seg_for(nmax)) {
    case 16: QAP_SEG(16);
    case 32: QAP_SEG(32);
    default: QAP_SEG(64);
    }
#undef QAP_SEG
}

template <int PM>
hipError_t Ops<PM>::inherit(qap_rlt2* ph, int pk, qap_rlt2* ch, const int* dfix)
{
    using T = StoreT<PM>;
    const Inst& P = ph->inst[pk];
    ChildSrc<T> src;
    src.B = static_cast<const T*>(ph->dB) + P.offB;
    src.C = static_cast<const T*>(ph->dC) + P.offC;
    src.D = ph->level == 2 ? static_cast<const T*>(ph->dD) + P.offD : nullptr;
    src.lb = ph->dLB + 2 * pk;
    src.N = P.N;
    src.mode = ph->dmode;
    src.ldD = P.ldD;
    src.fix = dfix;
    const int K = ch->K, M = P.N - 1;
    hipStream_t st = ch->stream;
    hipError_t e = in_launches(groups_of((long long)K * M * M, 256), 256, [&](long long first, unsigned grid) {
        hipLaunchKernelGGL((k_child_B<PM>), dim3(grid), dim3(256), 0, st, src, static_cast<T*>(ch->dB), ch->dLB,
                           ch->dInst, K, first);
        return hipGetLastError();
    });
    if (e != hipSuccess) return e;
    const long long perC = (long long)M * M * (M - 1) * (M - 1);
    const unsigned blocksC = (unsigned)groups_of(perC, 256);
    e = in_launches((long long)K * blocksC, 256, [&](long long first, unsigned grid) {
        hipLaunchKernelGGL((k_child_C<PM>), dim3(grid), dim3(256), 0, st, src, static_cast<T*>(ch->dC), ch->dInst,
                           blocksC, first);
        return hipGetLastError();
    });
    if (e != hipSuccess || ch->level == 1) return e;
    const Inst& I0 = ch->inst[0];
    T* D = static_cast<T*>(ch->dD);
    // Children of one size are packed with 128-byte aligned starts; the kernels
    // index each child's entries from its own offD.
    if (ch->dmode == kAllBlocks) {
        const long long perD = perC * I0.ldD;
        return in_launches(groups_of(K * perD, 256), 256, [&](long long first, unsigned grid) {
            hipLaunchKernelGGL((k_child_D<PM>), dim3(grid), dim3(256), 0, st, src, D, ch->dInst, K, perD, first);
            return hipGetLastError();
        });
    } else {
        const unsigned runs = (unsigned)(M * (M - 1) / 2 * (M - 2));
        const long long perD = (perC / 2) * (M - 2) * (M - 2);
        return in_launches((long long)K * runs, 256, [&](long long first, unsigned grid) {
            hipLaunchKernelGGL((k_child_runs<PM>), dim3(grid), dim3(256), 0, st, src, D, ch->dInst, runs,
                               (int)(ch->totalD / K - perD), first);
            return hipGetLastError();
        });
    }
}

}  // namespace qap
