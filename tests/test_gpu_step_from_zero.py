"""kl_step's fused pass onto cleared tendencies in every configuration that takes
the grid, and in place of one that does not: state and tendencies bitwise those
of zeroed arrays, kl_advec_u, kl_diff_uvw and kl_euler."""
import json

import numpy as np
import pytest
import torch

from paper_2303_12374_amd import inputs

pytestmark = pytest.mark.gpu


@pytest.fixture()
def m():
    from paper_2303_12374_amd import kl
    yield kl
    kl.kl_set_wisdom_dir(None)


VISC, DT = 1e-3, 2e-3


def start(m, dtype, shape, bc, layout):
    """Grid, fields, and fields and tendencies after a step of separate calls."""
    m.kl_set_wisdom_dir("/nonexistent")
    g = m.Grid(*shape, dtype=dtype, bc=bc, layout=inputs.plain_layout(*shape) if layout == "plain" else None)
    f = [g.full() for _ in range(3)]
    m.kl_generate_fields(g, 8, *f)
    m.kl_fill_ghosts(g, *f)
    rf, rt = [x.clone() for x in f], [g.zeros_interior(fill=-5.0) for _ in range(3)]
    m.kl_advec_u(g, rt[0], *rf)
    m.kl_diff_uvw(g, *rt, *rf, VISC)
    m.kl_euler(g, DT, *rf, *rt)
    return g, f, rf + rt


def compare(m, tmp_path, g, f, want, i):
    """One kl_step with configuration i selected, from NaN tendencies."""
    name = m.kl_variant_name(m.ADVEC_DIFF, g.dtype, i)
    (tmp_path / "advec_diff.wisdom").write_text(json.dumps(
        {"kernel": "advec_diff", "dtype": "f32" if g.dtype == 0 else "f64",
         "problem_size": [g.itot, g.jtot, g.ktot], "variant": name, "device": "forced", "arch": "gfx950",
         "time_ms": 1.0}) + "\n")
    m.kl_set_wisdom_dir(str(tmp_path))
    x, t = [a.clone() for a in f], [g.full(-5.0) for _ in range(3)]
    for a in t:
        g.interior(a).fill_(float("nan"))
    assert m.kl_selected_variant(g, m.ADVEC_DIFF) == i
    ok = m.kl_variant_eligible(g, m.ADVEC_DIFF, i, x + t)
    m.kl_step(g, VISC, DT, *x, *t)
    for a, b in zip(x + t, want):
        assert np.array_equal(a.cpu().numpy(), b.cpu().numpy(), equal_nan=True), name
    return ok


@pytest.mark.parametrize("bc", [0, 1, 2], ids=["zerograd", "nopen", "zperiodic"])
@pytest.mark.parametrize("dtype", [0, 1], ids=["f32", "f64"])
def test_every_eligible_configuration_runs_itself(m, tmp_path, dtype, bc):
    g, f, want = start(m, dtype, (256, 21, 19), bc, "padded")
    t = [g.full(0.0) for _ in range(3)]
    n = m.kl_num_variants(m.ADVEC_DIFF, dtype)
    eligible = [i for i in range(n) if m.kl_variant_eligible(g, m.ADVEC_DIFF, i, f + t)]
    # rows of 256 points are 64 chunks in FP32 and 128 in FP64, which rf_t256 does not take
    refused = {m.kl_variant_name(m.ADVEC_DIFF, dtype, i) for i in range(n)} - \
        {m.kl_variant_name(m.ADVEC_DIFF, dtype, i) for i in eligible}
    assert refused == (set() if dtype == 0 else {"rf_t256"})
    assert sum(compare(m, tmp_path, g, f, want, i) for i in eligible) == len(eligible)


@pytest.mark.parametrize("layout", ["padded", "plain"])
@pytest.mark.parametrize("dtype", [0, 1], ids=["f32", "f64"])
def test_refused_configuration_is_replaced(m, tmp_path, dtype, layout):
    """70 (FP64: 71) points are no whole number of vectors: such a selection runs
    another configuration with the same result."""
    g, f, want = start(m, dtype, (70 + dtype, 9, 11), 1, layout)
    t = [g.full(0.0) for _ in range(3)]
    refused = [i for i in range(m.kl_num_variants(m.ADVEC_DIFF, dtype))
               if not m.kl_variant_eligible(g, m.ADVEC_DIFF, i, f + t)]
    assert len(refused) > 10
    for i in refused:
        assert not compare(m, tmp_path, g, f, want, i)
