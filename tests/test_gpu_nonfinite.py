"""Infinite cache values and NaN queries: a value of +-inf under a positive
softmax weight makes its output dimension +-inf and leaves every other one
alone, however many partials a row has; a NaN query reaches no other row
(MI355X only)."""
import numpy as np
import pytest

import oracle
import paper_2403_08845_amd as bif
import workloads

from .parity import assert_parity
from .test_gpu_switch import run_path

pytestmark = pytest.mark.gpu

INF, MINUS_INF = 0x7F80, 0xFF80  # bf16 bit patterns

# Context partials of a row; with the four decode partials beside them: loads of
# the combine that are full and partly filled, for either kind, in its first 64
# partials and after them.
SPLITS = [1, 2, 3, 5, 31, 61, 63, 65]


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("b", [3, 24], ids=["few_rows", "many_rows"])
@pytest.mark.parametrize("splits", SPLITS)
def test_infinite_values(splits, b, d, monkeypatch):
    h, g, keys, m_d = 8, 2, 128, 128
    m_c = keys * splits - 5
    monkeypatch.setenv("BIFATTN_CTX_KEYS", str(keys))
    x = workloads.make_inputs(b, h, g, d, m_c, m_d, seed=2300 + splits)
    x["Vc"][:, 0, 5] = MINUS_INF         # in the first context partial
    x["Vc"][:, m_c - 1, 3] = INF         # in the last one
    x["Vd"][0, :, 0, 7] = INF            # first sample: in the first decode partial,
    x["Vd"][0, :, 100, 9] = MINUS_INF    # and in the last
    with bif.Plan(b, h, g, d, m_c, m_d, path="bifurcated") as plan:
        info = plan.info()
        print(f"[case] inf splits={splits} b={b} d={d} {info}", flush=True)
        assert info["ctx_splits"] == splits and info["dec_splits"] == 4
    out = run_path(x, "bifurcated")
    ref = oracle.attention(**x)
    special = np.isinf(ref)
    assert special.sum() == 2 * b * h + 2 * h
    assert np.array_equal(out[special], ref[special])
    assert_parity(np.where(special, 0, out), np.where(special, 0, ref), f"inf {splits} {b} {d}", x=x)


@pytest.mark.parametrize("case", [
    # b, h, g, d, m_c, m_d, n, kv: few rows; many rows with four and eight waves
    (3, 8, 2, 128, 300, 40, 1, "bf16"),
    (3, 8, 2, 64, 300, 40, 1, "int4"),
    (40, 8, 2, 128, 700, 40, 1, "bf16"),
    (40, 8, 2, 64, 700, 40, 1, "bf16"),
    (50, 16, 2, 64, 9000, 40, 1, "int8"),
    (40, 4, 2, 64, 900, 40, 2, "bf16"),
], ids=lambda c: "b%d_h%d_g%d_d%d_mc%d_md%d_n%d_%s" % c)
@pytest.mark.parametrize("path", ["standard", "bifurcated"])
def test_a_nan_query_stays_in_its_rows(case, path):
    b, h, g, d, m_c, m_d, n, kv = case
    x = workloads.make_inputs(b, h, g, d, m_c, m_d, seed=2400 + m_c, n=n, kv=kv)
    ref = oracle.attention(**x)
    x["q"] = x["q"].copy()
    x["q"][1] = 0x7FC0           # a whole sample
    x["q"][b - 1, 0, ..., 5] = 0x7FC0  # one element of one head
    bad = np.zeros(ref.shape, bool)
    bad[1] = bad[b - 1, 0] = True
    print(f"[case] nan query {case} {path}", flush=True)
    out = run_path(x, path)
    assert np.isnan(out[bad]).all()
    assert_parity(np.where(bad, 0, out), np.where(bad, 0, ref), f"nan query {case}", x=x)
