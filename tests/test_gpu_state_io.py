"""State I/O on the GPU: qap_rlt2_load_state, the FP64 certification cascade
on states with negative entries, and snapshot/restore.

The cascade is checked against a host FP64 computation written here from its
definition (c~ = c + (N-2) min(0, min D_beta), b~ = b + (N-1) min(0, min
C~_ij), LB + N min(0, min b~)), and against brute force: the certified bound
never exceeds the smallest represented objective over all permutations.
"""
import numpy as np
import pytest

import qapgen
from oracle import brute
from paper_1510_02065_amd import QapError, Rlt2
from tests import layout

pytestmark = pytest.mark.gpu
PRECISIONS = ["fp64", "fp32", "fp32n"]


def _host_cascade(N, lb, B, C, D):
    n1, n2 = N - 1, N - 2
    md = np.minimum(0.0, D.reshape(-1, n2 * n2).min(axis=1))
    ct = C + n2 * md
    mc = np.minimum(0.0, ct.reshape(N * N, n1 * n1).min(axis=1))
    bt = B + n1 * mc
    return lb + N * min(0.0, bt.min())


@pytest.mark.parametrize("precision", PRECISIONS)
def test_load_state_round_trip(precision):
    F, D = qapgen.small(8, 3)
    g = Rlt2(F, D, precision=precision)
    g.ascend(2)
    lb, B, C, Dst = g.read_state()
    h = Rlt2(F, D, precision=precision)
    h.load_state(0, lb, B, C, Dst)
    lb2, B2, C2, D2 = h.read_state()
    assert lb2 == lb
    np.testing.assert_array_equal(B2, B)
    np.testing.assert_array_equal(C2, C)
    np.testing.assert_array_equal(D2, Dst)
    # Both continue identically from the same state.
    g.ascend(2)
    h.ascend(2)
    for x, y in zip(g.read_state(), h.read_state()):
        np.testing.assert_array_equal(x, y)
    g.close()
    h.close()


@pytest.mark.parametrize("precision", PRECISIONS)
@pytest.mark.parametrize("complementary", [True, False])
def test_certify_with_negative_entries(precision, complementary):
    F, D = qapgen.small(8, 5)
    N = 8
    print(f"cascade {precision} complementary={complementary}", flush=True)
    g = Rlt2(F, D, precision=precision, complementary=complementary)
    g.ascend(2)
    lb, B, C, Dst = g.read_state()
    rng = np.random.default_rng(11)
    n2 = N - 2
    nblk = N * N * (N - 1) ** 2
    # Plant negative entries: in D blocks (both blocks of a complementary
    # pair, which are stored once), in C and in B; magnitudes chosen so that
    # every level of the cascade contributes.
    Dn = Dst.reshape(nblk, n2 * n2).copy()
    I, J, K, Nn = layout.c_index_arrays(N)
    pos = {(int(I[x]), int(J[x]), int(K[x]), int(Nn[x])): x for x in range(nblk)}
    for beta in rng.choice(nblk, 40, replace=False):
        i, j, k, n = int(I[beta]), int(J[beta]), int(K[beta]), int(Nn[beta])
        twin = pos[(k, n, i, j)]
        e = rng.integers(0, n2 * n2)
        v = -float(rng.uniform(0.5, 20.0))
        Dn[beta, e] = v
        Dn[twin, e] = v
    Cn = C.copy()
    Cn[rng.choice(C.size, 30, replace=False)] -= rng.uniform(50.0, 400.0, 30)
    Bn = B.copy()
    Bn[rng.choice(B.size, 5, replace=False)] -= rng.uniform(100.0, 900.0, 5)
    g.load_state(0, lb, Bn, Cn, Dn.ravel())
    lb2, B2, C2, D2 = g.read_state()   # as stored (FP32 modes rounded once)
    cert = g.certify()
    ref = _host_cascade(N, lb2, B2, C2, D2)
    assert cert < lb2                     # the corrections ran
    assert cert <= ref + 1e-12 * abs(ref)  # directed rounding only lowers it
    assert cert == pytest.approx(ref, rel=1e-12, abs=1e-9)
    # Validity against brute force: every permutation's represented objective
    # is at least the certified bound.
    perms = brute.all_perms(N)
    rep = layout.represented(N, lb2, B2, C2, D2, perms)
    assert cert <= rep.min() + 1e-9 * abs(rep.min())
    g.close()


@pytest.mark.parametrize("complementary", [True, False])
def test_certified_sweep_rounds_down_with_negative_entries(complementary):
    """Steps 1-3 in certified FP32 on a loaded state holding negative entries
    (the six-way means then take the directed path for terms of either sign):
    every member of every six-way group must end at or below the exact mean
    of (member + spread share of its block), computed here in rational
    arithmetic from the stored floats, and within a few FP32 steps of it."""
    from fractions import Fraction
    F, D = qapgen.small(8, 5)
    N, n1, n2 = 8, 7, 6
    g = Rlt2(F, D, precision="fp32", complementary=complementary)
    g.ascend(2)
    lb, B, C, Dst = g.read_state()
    rng = np.random.default_rng(12)
    nblk = N * N * n1 * n1
    I, J, K, Nn = layout.c_index_arrays(N)
    pos = {(int(I[x]), int(J[x]), int(K[x]), int(Nn[x])): x for x in range(nblk)}
    Dn = Dst.reshape(nblk, n2 * n2).copy()
    for beta in rng.choice(nblk, 60, replace=False):
        i, j, k, n = int(I[beta]), int(J[beta]), int(K[beta]), int(Nn[beta])
        e = rng.integers(0, n2 * n2)
        v = -float(rng.uniform(0.5, 40.0))
        Dn[beta, e] = v
        Dn[pos[(k, n, i, j)], e] = v     # the complementary block's same entry
    Cn = C.copy()
    Cn[rng.choice(C.size, 40, replace=False)] -= rng.uniform(5.0, 200.0, 40)
    Bn = B.copy()
    Bn[rng.choice(B.size, 6, replace=False)] -= rng.uniform(50.0, 500.0, 6)
    g.load_state(0, lb, Bn, Cn, Dn.ravel())
    _, B2, C2, D2 = g.read_state()        # the stored floats
    g.step(3)
    _, B3, C3, D3 = g.read_state()
    g.close()
    assert not B3.any() and not C3.any()  # both spread onward and cleared
    D2 = D2.reshape(nblk, n2 * n2)
    D3 = D3.reshape(nblk, n2 * n2)
    assert (D2 < 0).any()

    def beta_of(a, la, b, lb_):
        return ((a * N + la) * n1 + (b - (b > a))) * n1 + (lb_ - (lb_ > la))

    def entry(a, la, b, lb_, c, lc):
        return (c - (c > a) - (c > b)) * n2 + (lc - (lc > la) - (lc > lb_))

    share = {}
    def share_of(bt):
        if bt not in share:
            i, j = int(I[bt]), int(J[bt])
            share[bt] = (Fraction(float(C2[bt])) + Fraction(float(B2[i * N + j])) / n1) / n2
        return share[bt]

    checked = signed = 0
    worst = 0.0
    for f0 in range(N):
        for f1 in range(f0 + 1, N):
            for f2 in range(f1 + 1, N):
                for l0 in range(N):
                    for l1 in range(N):
                        if l1 == l0:
                            continue
                        for l2 in range(N):
                            if l2 == l0 or l2 == l1:
                                continue
                            P = ((f0, l0), (f1, l1), (f2, l2))
                            members = []
                            for a, b, c in ((0, 1, 2), (0, 2, 1), (1, 0, 2), (1, 2, 0), (2, 0, 1), (2, 1, 0)):
                                bt = beta_of(P[a][0], P[a][1], P[b][0], P[b][1])
                                e = entry(P[a][0], P[a][1], P[b][0], P[b][1], P[c][0], P[c][1])
                                members.append((bt, e))
                            terms = [Fraction(float(D2[bt, e])) + share_of(bt) for bt, e in members]
                            mean = sum(terms) / 6
                            got = {float(D3[bt, e]) for bt, e in members}
                            assert len(got) == 1, "members of one group differ"
                            v = got.pop()
                            assert Fraction(v) <= mean, (P, v, float(mean))
                            scale = max(abs(float(t)) for t in terms) + abs(float(mean))
                            gap = float(mean - Fraction(v))
                            assert gap <= 4 * 2.0 ** -23 * scale, (P, v, float(mean), gap)
                            worst = max(worst, gap / scale if scale else 0.0)
                            checked += 1
                            signed += any(float(D2[bt, e]) < 0 or share_of(bt) < 0 for bt, e in members)
    print(f"certified sweep: {checked} groups, {signed} with a negative term, worst gap {worst:.2e} of the scale",
          flush=True)
    assert signed > 0


def test_load_state_rejects_bad_input():
    F, D = qapgen.small(8, 0)
    g = Rlt2(F, D)
    lb, B, C, Dst = g.read_state()
    B[3] = np.nan
    with pytest.raises(QapError):
        g.load_state(0, lb, B, None, None)
    with pytest.raises(QapError):
        g.load_state(1, lb, None, None, None)   # one instance only
    g.close()


@pytest.mark.parametrize("precision", PRECISIONS)
def test_snapshot_restore_is_bitwise_continuation(precision):
    F, D = qapgen.uniform(12, 1)
    print(f"snapshot {precision}", flush=True)
    ref = Rlt2(F, D, precision=precision, trace_level=2)
    ref.ascend(7)
    a = Rlt2(F, D, precision=precision, trace_level=2)
    a.ascend(3)
    snap = a.snapshot()
    a.close()   # the run is "killed" after 3 iterations
    b = Rlt2(F, D, precision=precision, trace_level=2)
    b.restore(snap)
    assert b.bound()[1] == 3
    b.ascend(4)
    for x, y in zip(ref.read_state(), b.read_state()):
        np.testing.assert_array_equal(x, y)
    for x, y in zip(ref.trace(), b.trace()):
        np.testing.assert_array_equal(x, y)
    np.testing.assert_array_equal(ref.lap_values()[0], b.lap_values()[0])
    assert b.bound() == ref.bound()
    ref.close()
    b.close()


def test_snapshot_batch_and_mismatch():
    F, D, fixes = qapgen.nodes(count=6, parent_N=12, seed=3, m_lo=2, m_hi=5)
    from paper_1510_02065_amd import subproblem
    nodes = [subproblem(F, D, fac, loc) for fac, loc in fixes]
    args = ([n[0] for n in nodes], [n[1] for n in nodes], [n[2] for n in nodes], [n[3] for n in nodes])
    ref = Rlt2.batch(*args)
    ref.ascend(5)
    a = Rlt2.batch(*args)
    a.ascend(2)
    snap = a.snapshot()
    b = Rlt2.batch(*args)
    b.restore(snap)
    b.ascend(3)
    np.testing.assert_array_equal(ref.bounds(), b.bounds())
    for k in range(len(nodes)):
        for x, y in zip(ref.read_state_k(k), b.read_state_k(k)):
            np.testing.assert_array_equal(x, y)
    other = Rlt2(*qapgen.small(8, 0))
    with pytest.raises(QapError):
        other.restore(snap)   # different instances
    with pytest.raises(QapError):
        b.restore(snap[:-9])  # truncated
    for h in (ref, a, b, other):
        h.close()


# Stretches of the streaming minimum over the stored blocks: one block row
# (N = 3), a stretch longer than the pair's locations (4, 12), exactly whole
# stretches and a short last one (18, 20).
@pytest.mark.parametrize("N,precision", [(3, "fp64"), (4, "fp32"), (12, "fp64"), (18, "fp32n"), (20, "fp64")])
def test_certify_finds_every_blocks_minimum(N, precision):
    F, D = qapgen.uniform(N, 2)
    g = Rlt2(F, D, precision=precision)
    rng = np.random.default_rng(N)
    n1, n2 = N - 1, N - 2
    I, J, K, Nn = layout.c_index_arrays(N)
    twin = ((K * N + Nn) * n1 + I - (I > K)) * n1 + J - (J > Nn)
    keep = I < K
    # One negative entry per stored block, at a random place; each block's in
    # turn is by far the smallest, so a block left out changes the bound.
    Dn = np.zeros((len(I), n2 * n2))
    C = np.zeros(len(I))
    B = np.zeros(N * N)
    stored = np.flatnonzero(keep)
    Dn[stored, rng.integers(0, n2 * n2, size=len(stored))] = -1.0 / 1024
    Dn[twin[stored]] = Dn[stored]
    for beta in rng.choice(stored, min(6, len(stored)), replace=False):
        X = Dn.copy()
        X[beta, rng.integers(0, n2 * n2)] = -64.0
        X[twin[beta]] = X[beta]
        g.load_state(0, 0.0, B, C, X.ravel())
        assert g.certify() == pytest.approx(_host_cascade(N, 0.0, B, C, X.ravel()), rel=1e-12)
    g.close()


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
def test_handles_after_a_closed_one_start_clean(precision):
    # A new handle may get the memory of one closed before it: of its own size,
    # a little larger, or another precision's.  Its results are those of the
    # first handle of the process, also with handles open side by side and from
    # several threads.
    import threading
    F, D = qapgen.small(12, 3)
    F11, D11 = qapgen.small(11, 4)

    def run(f, d, prec=precision):
        with Rlt2(f, d, precision=prec) as g:
            g.ascend(3)
            return (g.trace()[0], *g.read_state()[1:])

    first, other = run(F, D), run(F11, D11)
    run(F, D, "fp32n" if precision == "fp64" else "fp64")
    with Rlt2(F, D, precision=precision) as g:
        g.ascend(2)
        again, other2 = run(F, D), run(F11, D11)
        g.ascend(1)
        beside = (g.trace()[0], *g.read_state()[1:])
    from_threads = [None] * 4

    def work(i):
        for _ in range(5):
            from_threads[i] = run(F, D) if i % 2 else run(F11, D11)

    threads = [threading.Thread(target=work, args=(i,)) for i in range(4)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    for got, want in [(again, first), (other2, other), (beside, first), (from_threads[0], other),
                      (from_threads[1], first), (from_threads[2], other), (from_threads[3], first)]:
        for x, y in zip(got, want):
            np.testing.assert_array_equal(x, y)


def test_restore_refuses_a_configuration_that_cannot_hold_the_problems():
    # The snapshot's (lanes, columns) of every class: one of a kernel that
    # exists, with room for the class's problems, within a workgroup's LDS.
    F, D = qapgen.small(8, 2)   # one class in use per family, of 8 lanes
    g = Rlt2(F, D, trace_level=0)
    g.ascend(2)
    snap = g.snapshot()
    before = g.read_state()
    # From the end: per instance the iteration count and the length of the
    # trace (no entries at this level), before them 3 families x 4 classes x 2.
    at = len(snap) - 16 - 3 * 4 * 2 * 4
    cfg = np.frombuffer(snap[at:at + 96], dtype=np.int32).reshape(3, 4, 2)
    assert (cfg[:, 0] == [8, 1]).all()
    for f in range(3):
        for lanes, columns in [(4, 2), (8, 7), (16, 5), (64, 2), (0, 0), (-8, -1)]:
            bad = cfg.copy()
            bad[f, 0] = lanes, columns
            with pytest.raises(QapError) as e:
                g.restore(snap[:at] + bad.tobytes() + snap[at + 96:])
            assert e.value.status == -1, (f, lanes, columns)
    for x, y in zip(before, g.read_state()):
        np.testing.assert_array_equal(x, y)
    wider = cfg.copy()   # what an earlier build may have chosen
    wider[:, 0] = [[8, 2], [16, 1], [8, 8]]
    g.restore(snap[:at] + wider.tobytes() + snap[at + 96:])
    g.ascend(1)
    h = Rlt2(F, D, trace_level=0)
    h.ascend(3)
    for x, y in zip(h.read_state(), g.read_state()):
        np.testing.assert_array_equal(x, y)
    big = Rlt2(*qapgen.uniform(24, 1), trace_level=0)   # 32-lane classes
    snap = big.snapshot()
    cfg = np.frombuffer(snap[-16 - 96:-16], dtype=np.int32).reshape(3, 4, 2).copy()
    assert (cfg[:, 2] == [32, 1]).all()
    cfg[0, 2] = 16, 1   # 16 columns for problems of 22
    with pytest.raises(QapError):
        big.restore(snap[:-16 - 96] + cfg.tobytes() + snap[-16:])
    for x in (g, h, big):
        x.close()


def _free_bytes():
    torch = pytest.importorskip("torch")
    torch.cuda.synchronize()
    return torch.cuda.mem_get_info()[0]


def test_a_reused_block_counts_at_its_real_size():
    # Batches whose D shrinks by about a tenth from one to the next: each may
    # use the memory of one closed before it, but none may hold more than a
    # quarter beyond its own need.
    F, D = qapgen.uniform(16, 1)
    one = 16 ** 2 * 15 ** 2 * 14 ** 2 // 2 * 8   # bytes of an instance's D
    Rlt2(F, D).close()
    Rlt2(*qapgen.small(8, 0)).close()   # next to nothing is kept now
    free = _free_bytes()
    for count in (10, 9, 8):
        for _ in range(3):
            Rlt2.batch([F] * count, [D] * count).close()
    g = Rlt2.batch([F] * 7, [D] * 7)
    held = free - _free_bytes()
    g.close()
    print(f"held {held / one:.2f} instances' D for 7", flush=True)
    assert held <= 1.25 * 7 * one + 0.6 * one   # the rest: B, C, the trace and the allocator's granularity


def test_closing_gives_the_memory_back():
    # A handle's memory is free again once it is closed.  One that is opened and
    # closed again and again at one size may keep its D's between two of them,
    # until the program asks for it back.
    from paper_1510_02065_amd import release_memory
    F, D = qapgen.uniform(24, 1)
    one = 24 ** 2 * 23 ** 2 * 22 ** 2 // 2 * 8   # 590 MB
    Rlt2(*qapgen.small(8, 0)).close()
    release_memory()
    free = _free_bytes()
    with Rlt2(F, D) as g:
        g.ascend(1)
        assert _free_bytes() <= free - one
    assert _free_bytes() >= free - one // 8
    for _ in range(4):
        Rlt2(F, D).close()
    release_memory()
    assert _free_bytes() >= free - one // 8
    release_memory()   # nothing kept: nothing happens
