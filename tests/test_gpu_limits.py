"""The size limits of one handle on one MI355X.

* N = 64, the largest size (one wave64 lane per column of the C->B and
  B->LB problems), in FP32 round-to-nearest: 125 GB of stored D.  The oracle's
  dense state would need 550 GB, so this size is checked by what holds at any
  size: iteration 0 is the Gilmore-Lawler bound (computed here with the
  oracle's assignment solver), the bound does not fall, stays below the
  objective of the B-level assignment improved by pairwise exchanges, and the
  reduced costs stay >= 0.
* A state that cannot fit in HBM (N = 64 in FP64 with every block stored:
  500 GB) is refused with QAP_ENOMEM before anything is allocated.
* Batches with more work per step than one launch may have threads (2^32).
"""
import numpy as np
import pytest

import oracle
import qapgen
from oracle import brute
from paper_1510_02065_amd import QapError, Rlt2, local_search
from paper_1510_02065_amd import _binding as B

pytestmark = pytest.mark.gpu


def test_state_larger_than_hbm_is_refused():
    F, D = qapgen.clustered(64, 0)
    with pytest.raises(QapError) as e:
        Rlt2(F, D, precision="fp64", complementary=False)
    assert e.value.status == B.QAP_ENOMEM


def test_maximum_size_n64_fp32_nearest():
    F, D = qapgen.clustered(64, 0)
    print("N=64 FP32 nearest: create", flush=True)
    g = Rlt2(F, D, precision="fp32n")
    glb = brute.gilmore_lawler(F, D, lap=lambda L: oracle.lap_solve(L)[0])
    lb0 = g.bound()[0]
    assert lb0 == pytest.approx(glb, rel=1e-5)
    print("N=64 FP32 nearest: one iteration", flush=True)
    lb1 = g.ascend(1)
    assert lb1 >= lb0 * (1 - 1e-6)
    perm, ub = local_search(F, D, g.assignment(0))
    assert sorted(perm.tolist()) == list(range(64))
    assert lb1 <= ub * (1 + 1e-5)
    _, Bst, Cst, _ = g.read_state(want_D=False)
    assert Bst.min() >= 0 and Cst.min() >= 0
    print(f"N=64: GLB {glb:.6g}, LB_0 {lb0:.6g}, LB_1 {lb1:.6g}, UB {ub:.6g}", flush=True)
    g.close()


def _same_bounds(g, F, D, iters, **kw):
    h = Rlt2(F, D, **kw)
    h.ascend(iters)
    g.ascend(iters)
    np.testing.assert_array_equal(g.bounds(), h.bounds()[0])
    last = len(g.Ns) - 1
    for x, y in zip(g.read_state_k(last, want_D=False), h.read_state(want_D=False)):
        np.testing.assert_array_equal(x, y)
    h.close()


def test_level1_batch_of_more_pairs_than_one_launch():
    # 306000 instances of N = 11: 16.8 million facility pairs, a workgroup of
    # 256 threads each.
    F, D = qapgen.small(11, 3)
    count = 306000
    print("level 1, 306000 instances", flush=True)
    with Rlt2.batch([F] * count, [D] * count, precision="fp32n", level=1) as g:
        _same_bounds(g, F, D, 2, precision="fp32n", level=1)


def test_level1_batch_of_more_entries_than_one_launch():
    # 360000 instances of N = 11: 4.4 billion entries of C, a thread each in the
    # single step 1 and in the certification.
    F, D = qapgen.small(11, 5)
    count = 360000
    print("level 1, 360000 instances", flush=True)
    with Rlt2.batch([F] * count, [D] * count, precision="fp32", level=1) as g, \
            Rlt2(F, D, precision="fp32", level=1) as h:
        for s in (3, 5, 6, 7):
            g.step(s)
            h.step(s)
        for x, y in zip(g.bounds(certified=True), h.bounds(certified=True)):
            np.testing.assert_array_equal(x, y[0])


# 45000 instances of N = 11: 272 million blocks of D, 16 lanes each; 52000 of
# them: 8.6 million facility triples, 512 threads each.
@pytest.mark.parametrize("count", [45000, 52000])
def test_level2_batch_of_more_assignments_than_one_launch(count):
    F, D = qapgen.small(11, 4)
    print(f"level 2, {count} instances", flush=True)
    with Rlt2.batch([F] * count, [D] * count, precision="fp32n") as g:
        _same_bounds(g, F, D, 2, precision="fp32n")
        lb, cert = g.bounds(certified=True)
        assert (cert == cert[0]).all() and cert[0] <= lb[0]


def test_lap_batch_of_more_problems_than_one_launch():
    # 67.2 million problems, 100000 of 33 rows and the others of one: the launch
    # of the largest size class has a wave per problem of the batch.
    torch = pytest.importorskip("torch")
    from paper_1510_02065_amd import lap_solve_device
    count, large, n = 67200000, 100000, 33
    dev = torch.device("cuda:0")
    M = qapgen.random_matrix(n, 1, "int")
    sizes = torch.ones(count, dtype=torch.int32, device=dev)
    sizes[:large] = n
    entries = sizes.long() ** 2
    at = torch.cumsum(entries, 0) - entries
    small = torch.arange(count - large, device=dev) % 1000
    cost = torch.cat([torch.tensor(M.ravel(), device=dev).repeat(large), small.double()]).float()
    value = torch.full((count,), -1.0, dtype=torch.float64, device=dev)
    print(f"{count} assignment problems", flush=True)
    lap_solve_device(sizes, at, None, cost, value, fp32=True, nearest=True, stream=torch.cuda.current_stream())
    torch.cuda.synchronize()
    assert bool((value[large:] == small).all())
    want = oracle.lap_concentrate(M)[0]
    assert float(value[:large].min()) == float(value[:large].max())
    assert abs(float(value[0]) - want) <= 1e-5 * want


def test_children_of_more_runs_than_one_launch():
    # 600000 children of N = 5: 18 million runs, a workgroup of 256 threads each.
    F, D = qapgen.small(6, 3)
    with Rlt2(F, D, trace_level=0) as g:
        g.ascend(2)
        count = 600000
        fac = np.arange(count, dtype=np.int32) % 6
        loc = np.arange(count, dtype=np.int32) // 6 % 6
        print("600000 children", flush=True)
        few = g.children(0, fac[:36], loc[:36])
        with g.children(0, fac, loc) as ch:
            for c in (0, 35, 36 * 8000 + 7, count - 1):
                for x, y in zip(ch.read_state_k(c), few.read_state_k(c % 36)):
                    np.testing.assert_array_equal(x, y)
        few.close()
