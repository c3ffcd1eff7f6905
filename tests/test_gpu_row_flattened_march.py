"""Long marches of the row-flattened tiles, where the register ring wraps and
the LDS planes rotate past the unrolled levels: both types, every boundary mode,
remainders of levels, tendencies cached and streamed, single launches, batches
and served steps with eight levels a tile and more.  Bitwise against configuration 0."""
import json

import numpy as np
import pytest
import torch

from paper_2303_12374_amd import inputs
from test_gpu_row_flattened import run

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True)
def no_wisdom(tmp_path):
    from paper_2303_12374_amd import kl as m
    m.kl_set_wisdom_dir(str(tmp_path / "wisdom"))
    yield
    m.kl_set_wisdom_dir(None)


# 10 to 29 levels a tile; the last two of each type stream diff_uvw's, then also
# advec_u's tendencies
@pytest.mark.parametrize("bc", [0, 1, 2], ids=["zerograd", "nopen", "zperiodic"])
@pytest.mark.parametrize("dtype,size,ran", [(0, (301, 203, 65), 8), (0, (97, 301, 41), 8), (0, (520, 205, 105), 4),
                                            (0, (640, 203, 126), 4), (1, (150, 201, 66), 8), (1, (301, 203, 92), 4),
                                            (1, (160, 256, 141), 8), (1, (331, 203, 131), 4)])
def test_long_marches_bitwise_equal_default(dtype, size, ran, bc):
    from paper_2303_12374_amd import kl as m
    g = m.Grid(*size, dtype=dtype, bc=bc, layout=inputs.plain_layout(*size))
    assert run(m, g, dtype, ("rf_t256", "rf_t512")) == ran


@pytest.mark.parametrize("zero", [False, True], ids=["accumulate", "cleared"])
# more than one tile a slot (8 levels); as many slots as tiles of 16, of 32 levels
@pytest.mark.parametrize("dtype,shapes,levels", [
    (0, [(125, 1200, 43), (124, 1100, 44), (128, 1300, 41)], 8), (1, [(62, 1200, 43), (61, 1100, 44), (64, 1300, 41)], 8),
    (0, [(125, 300, 60), (124, 290, 63), (128, 360, 61)], 16), (1, [(62, 300, 60), (61, 290, 63), (64, 360, 61)], 16),
    (0, [(125, 600, 60), (124, 510, 63), (128, 520, 67)], 32), (1, [(62, 600, 60), (61, 510, 63), (64, 520, 67)], 32)])
def test_batch_of_long_tiles(dtype, shapes, levels, zero):
    from paper_2303_12374_amd import kl as m
    grids, fields, want = [], [], []
    for n, s in enumerate(shapes):
        g = m.Grid(*s, dtype=dtype, bc=n % 3)
        f = [g.full(0.0) for _ in range(3)]
        m.kl_generate_fields(g, 60 + n, *f)
        m.kl_fill_ghosts(g, *f)
        t = [g.zeros_interior(fill=-3.0) for _ in range(3)]
        for x in t:
            g.interior(x).fill_(0.0 if zero else 0.75)
        m.kl_launch_variant(g, m.ADVEC_DIFF, 0, f + t, 1e-3)
        grids.append(g)
        fields.append(f + [g.full(-3.0) for _ in range(3)])
        want.append(t)
    b = m.kl_batch_create(grids, fields, 1e-3, zero)
    try:
        (_, name, tiles), = m.kl_batch_groups(b)
        assert name == "rf_t256"
        rows = [256 // -(-s[0] // (4 if dtype == 0 else 2)) for s in shapes]
        assert tiles == sum(-(-s[1] // r) * -(-s[2] // levels) for s, r in zip(shapes, rows)) >= 256
        for _ in range(3):
            for g, f in zip(grids, fields):
                for x in f[3:]:
                    g.interior(x).fill_(0.75)
            torch.cuda.synchronize()
            m.kl_batch_run(b)
            torch.cuda.synchronize()
            for f, w in zip(fields, want):
                for x, y in zip(f[3:], w):
                    assert torch.equal(x, y)
    finally:
        m.kl_batch_destroy(b)


@pytest.mark.parametrize("dtype,size,bc", [(0, (128, 256, 68), 0), (0, (192, 256, 43), 2), (1, (96, 256, 43), 1),
                                           (1, (64, 512, 45), 0)])
def test_served_step_of_long_tiles(tmp_path, dtype, size, bc):
    from paper_2303_12374_amd import kl as m
    nsteps, dt, visc, seed = 3, 1e-3, 1e-5, 9
    g = m.Grid(*size, dtype=dtype, bc=bc)
    a, b = [g.full() for _ in range(3)], [g.full() for _ in range(3)]
    m.kl_generate_fields(g, seed, *a)
    m.kl_fill_ghosts(g, *a)
    for _ in range(nsteps):
        m.kl_launch_variant_dt(g, m.STEP, 0, a + b, visc, dt)
        a, b = b, a
    d = tmp_path / "rec"
    d.mkdir()
    (d / "step.wisdom").write_text(json.dumps({"kernel": "step", "dtype": "f32" if dtype == 0 else "f64",
                                               "problem_size": list(size), "variant": "rf_t256", "device": "forced",
                                               "arch": "gfx950", "time_ms": 1.0}) + "\n")
    m.kl_set_wisdom_dir(str(d))
    assert m.kl_variant_name(m.STEP, dtype, m.kl_selected_variant(g, m.STEP)) == "rf_t256"
    chunks = -(-size[0] // (4 if dtype == 0 else 2))
    assert -(-size[1] // (256 // chunks)) * -(-size[2] // 8) >= 256  # else four levels a tile
    arena = torch.empty(1 << 28, dtype=torch.uint8, device="cuda")
    h = m.kl_server_create(arena, arena.numel(), arena.numel())
    try:
        t = m.kl_submit(h, *size, dtype, bc, nsteps, dt, visc, seed)
        rc, res = m.kl_poll(h, t)
        while rc == m.ERR_AGAIN:
            rc, res = m.kl_poll(h, t)
        assert res.state == 2
        torch.cuda.synchronize()
        whole = arena.view(g.tdtype)
        for p, want in zip(res.fields, a):
            off = (p - arena.data_ptr()) // whole.element_size()
            got = whole.as_strided((size[2] + 2, size[1] + 2, size[0] + 2), (res.kstride, res.jstride, 1), off + res.off)
            assert np.array_equal(got.cpu().numpy(), g.box(want).cpu().numpy())
        m.kl_release(h, t)
    finally:
        m.kl_server_destroy(h)


# the arrays of all grids just within 256 MB, where tendencies stay in the caches, and just beyond
@pytest.mark.parametrize("dtype,size", [(0, (100, 100, 1066)), (0, (100, 100, 1067)), (1, (100, 100, 533)),
                                        (1, (100, 100, 534))], ids=str)
def test_batch_at_the_size_of_the_cache(dtype, size):
    from paper_2303_12374_amd import kl as m
    g = m.Grid(*size, dtype=dtype)
    f = [g.full(0.0) for _ in range(3)]
    m.kl_generate_fields(g, 5, *f)
    m.kl_fill_ghosts(g, *f)
    t, o = [g.full(0.5) for _ in range(3)], [g.full(0.5) for _ in range(3)]
    b = m.kl_batch_create([g], [f + o], 1e-3, False)
    try:
        assert m.kl_batch_groups(b)[0][1] == "rf_t256"
        for _ in range(2):
            m.kl_launch_variant(g, m.ADVEC_DIFF, 0, f + t, 1e-3)
            m.kl_batch_run(b)
            torch.cuda.synchronize()
            for x, y in zip(t, o):
                assert torch.equal(g.interior(x), g.interior(y))
    finally:
        m.kl_batch_destroy(b)
