"""kl_tune times the fused step as a program runs it: from one field set into
the other and back."""
import pytest
import torch

from paper_2303_12374_amd import inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("layout", ["padded", "plain"])
@pytest.mark.parametrize("dtype", [0, 1], ids=["f32", "f64"])
def test_step_is_tuned_on_two_field_sets_in_turn(tmp_path, dtype, layout):
    """The timed steps go on from each other's results, so what they leave in ut, vt,
    wt is several steps on; u, v, w, which the caller keeps, are not written."""
    from paper_2303_12374_amd import kl as m
    size = (40, 12, 10)
    g = m.Grid(*size, dtype=dtype, bc=2, layout=inputs.plain_layout(*size) if layout == "plain" else None)
    f = [g.full(0.25) for _ in range(3)]
    m.kl_generate_fields(g, 5, *f)
    m.kl_fill_ghosts(g, *f)
    before = [x.clone() for x in f]
    t = [g.full(-5.0) for _ in range(3)]
    try:
        res = m.kl_tune(g, f + t, m.TUNE_STEP, wisdom_dir=str(tmp_path), budget_s=20.0)
    finally:
        m.kl_set_wisdom_dir(None)
    assert len(res) > 1 and all(ms > 0 for _, ms in res)
    assert (tmp_path / "step.wisdom").exists()
    for a, b in zip(f, before):
        assert torch.equal(a, b)
    a, b = [x.clone() for x in f], [g.full(0.0) for _ in range(3)]
    states = []
    for _ in range(40):  # the tuner's viscosity and time step
        m.kl_launch_variant_dt(g, m.STEP, 0, a + b, 1e-5, 1e-4)
        states.append([g.box(x).clone() for x in b])
        a, b = b, a
    got = [g.box(x) for x in t]
    at = [n for n, s in enumerate(states) if all(torch.equal(x, y) for x, y in zip(got, s))]
    assert at and at[0] > 1
