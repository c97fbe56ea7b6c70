"""The steps 1-3 kernels for one stored block per complementary pair (one
workgroup per facility triple when the triple fits in LDS, boxes of
locations otherwise) against the every-block comparison path, at the sizes where the
choice changes: bit for bit after two iterations, on the trace and on every
concentration's value."""
import numpy as np
import pytest

import qapgen
from paper_1510_02065_amd import Rlt2

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N,precision", [(25, "fp64"), (26, "fp64"), (32, "fp32"), (33, "fp32")])
def test_stored_half_matches_every_block(N, precision):
    F, D = qapgen.clustered(N, 3)
    print(f"sweep paths N={N} {precision}", flush=True)
    a = Rlt2(F, D, precision=precision, trace_level=2, complementary=True)
    a.ascend(2)
    ta, va = a.trace()[0], a.lap_values()
    a.close()
    b = Rlt2(F, D, precision=precision, trace_level=2, complementary=False)
    b.ascend(2)
    tb, vb = b.trace()[0], b.lap_values()
    b.close()
    np.testing.assert_array_equal(ta, tb)
    for x, y in zip(va, vb):
        np.testing.assert_array_equal(x, y)


# Box edges of k_sweep_box: FP64 16 (two tiles, the last one short), 12 (three
# tiles, the last one short), 13 (whole); FP32 18, 22 (the largest), 15 (three tiles).
@pytest.mark.parametrize("N,precision", [(31, "fp64"), (34, "fp64"), (39, "fp64"), (36, "fp32n"), (44, "fp32"),
                                         (45, "fp32n")])
def test_box_sweep_matches_every_block(N, precision):
    test_stored_half_matches_every_block(N, precision)


@pytest.mark.parametrize("overlap", [True, False])
def test_batch_across_sweep_kernels_equals_individual_handles(overlap):
    # 27: boxes; 23: persistent per-triple; 16, 8: a workgroup per triple.
    cases = [qapgen.clustered(27, 1), qapgen.small(8, 1), qapgen.clustered(23, 1), qapgen.uniform(16, 1)]
    print("batch N =", [F.shape[0] for F, _ in cases], "overlap", overlap, flush=True)
    g = Rlt2.batch([F for F, _ in cases], [D for _, D in cases], trace_level=2, overlap=overlap)
    g.ascend(3)
    for k, (F, D) in enumerate(cases):
        h = Rlt2(F, D, trace_level=2)
        h.ascend(3)
        np.testing.assert_array_equal(h.trace()[0], g.trace_k(k)[0])
        for x, y in zip(h.lap_values(), g.lap_values_k(k)):
            np.testing.assert_array_equal(x, y)
        h.close()
    g.close()
