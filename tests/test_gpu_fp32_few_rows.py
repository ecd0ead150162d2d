"""GPU: the FP32 forward of few observables and many gates on both sides of the
line between the non-zero entries and the matrix cores: phases against the sum
that both stand for."""
import numpy as np
import pytest

import workloads as W
from paper_2501_04776_amd import api
from tests.gpu_util import DevWorkload
from tests.test_gpu_fp32_chain import _phases

pytestmark = pytest.mark.gpu


# C 4, 9 and 20 % full
@pytest.mark.parametrize("op_w", [1, 2, 6])
def test_fp32_few_observables_bitwise(op_w, monkeypatch):
    n, m, l, s, splits = 60, 100000, 52, 500, 13
    assert l * s * m >= 2 ** 31
    monkeypatch.setenv("IQP_FWD_SPLITS", str(splits))
    w = W.small_random(80 + op_w, n, m, l, s, gate_w=(1, 4), op_w=(op_w, op_w))
    dw = DevWorkload(w)
    circ = api.Circuit(n, dw.gens, dw.theta)
    _, _, ph = api.iqp_expval(circ, dw.ops, dw.samples, "fp32", phase_save=True)
    rows = [0, 25, 51]
    got = ph.cpu().numpy()[rows]
    ref = _phases(w, dw.ops01, rows, splits)
    # the last FP64 steps may round differently: one FP32 ulp of the phase
    assert (np.abs(got - ref) <= np.spacing(np.abs(got).astype(np.float32))).all()
    assert (got == ref.astype(np.float32)).mean() > 0.999
