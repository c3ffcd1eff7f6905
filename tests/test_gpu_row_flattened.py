"""Row-flattened configurations (rf_t256, rf_t512) where they can go wrong:
rows of one point, of one chunk, partial last chunks, rows that fill a block
in two or one halves, row blocks with a remainder, one and two levels per
tile, misaligned rows, all boundary modes; and a grid above the size from
which tendencies are streamed.  Each is compared bitwise, ghost and padding
cells included, with the default configuration (the fused step: with
configuration 0), which the oracle tests hold."""
import numpy as np
import pytest
import torch

from paper_2303_12374_amd import inputs

pytestmark = pytest.mark.gpu

SHAPES = [(1, 1, 2), (3, 5, 4), (5, 4, 6), (127, 40, 5), (301, 11, 9), (1023, 3, 3), (48, 300, 3), (160, 513, 2)]


def run(m, g, dtype, names):
    """{kernel: outputs of every configuration in names} from the same inputs."""
    f = [g.full(0.25) for _ in range(3)]
    m.kl_generate_fields(g, 31, *f)
    m.kl_fill_ghosts(g, *f)
    ran = 0
    for kernel in (m.ADVEC_U, m.DIFF_UVW, m.ADVEC_DIFF, m.STEP):
        ref = None
        for i in range(m.kl_num_variants(kernel, dtype)):
            name = m.kl_variant_name(kernel, dtype, i)
            if i and name not in names:
                continue
            out = [g.full(-5.0) for _ in range(3)]
            if not m.kl_variant_eligible(g, kernel, i, f + out):
                continue
            if kernel != m.STEP:
                for n, x in enumerate(out):
                    g.interior(x).fill_(0.5 + n)
            m.kl_launch_variant_dt(g, kernel, i, f + out, 1e-3, 2e-3)
            if ref is None:
                ref = out
                continue
            for a, b in zip(out, ref):
                assert torch.equal(a, b), (m.KERNEL_NAMES[kernel], name)
            ran += 1
    return ran


@pytest.mark.parametrize("layout", ["padded", "plain"])
@pytest.mark.parametrize("bc", [0, 1, 2], ids=["zerograd", "nopen", "zperiodic"])
@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: "x".join(map(str, s)))
@pytest.mark.parametrize("dtype", [0, 1], ids=["f32", "f64"])
def test_row_flattened_bitwise_equals_default(dtype, shape, bc, layout):
    from paper_2303_12374_amd import kl as m
    g = m.Grid(*shape, dtype=dtype, bc=bc, layout=inputs.plain_layout(*shape) if layout == "plain" else None)
    ran = run(m, g, dtype, ("rf_t256", "rf_t512"))
    chunks = -(-shape[0] // (4 if dtype == 0 else 2))
    assert ran == (8 if chunks <= 80 else 4 if chunks <= 256 else 0)


def test_row_flattened_streams_large_tendencies():
    from paper_2303_12374_amd import kl as m
    g = m.Grid(301, 256, 211, dtype=0)
    assert 4 * 4 * g.npoints > 256e6
    assert run(m, g, 0, ("rf_t256", "rf_t512")) == 8


@pytest.mark.parametrize("dtype", [0, 1], ids=["f32", "f64"])
def test_batch_of_odd_unpadded_grids(dtype):
    """Grids no aligned tile takes, in one batch, onto tendencies that are read
    and onto cleared ones, bitwise the separate launches."""
    from paper_2303_12374_amd import kl as m
    shapes = [(33, 7, 5), (1, 3, 4), (75, 40, 33), (127, 9, 70), (50, 50, 50), (200, 3, 2)]
    grids, fields, init = [], [], []
    for n, s in enumerate(shapes):
        g = m.Grid(*s, dtype=dtype, bc=n % 3, layout=inputs.plain_layout(*s))
        f = [g.full(0.0) for _ in range(3)]
        m.kl_generate_fields(g, 40 + n, *f)
        m.kl_fill_ghosts(g, *f)
        grids.append(g)
        fields.append(f + [g.full(-3.0) for _ in range(3)])
    for zero in (False, True):
        want = []
        for g, f in zip(grids, fields):
            t = [g.zeros_interior(fill=-3.0) for _ in range(3)]
            for x in t:
                g.interior(x).fill_(0.0 if zero else 0.75)
            m.kl_advec_u(g, t[0], *f[:3])
            m.kl_diff_uvw(g, *t, *f[:3], 1e-3)
            want.append([x.cpu().numpy() for x in t])
        b = m.kl_batch_create(grids, fields, 1e-3, zero)
        try:
            for _ in range(3):
                for g, f in zip(grids, fields):
                    for x in f[3:]:
                        g.interior(x).fill_(0.75)
                torch.cuda.synchronize()
                m.kl_batch_run(b)
                torch.cuda.synchronize()
                for f, w in zip(fields, want):
                    for x, y in zip(f[3:], w):
                        assert np.array_equal(x.cpu().numpy(), y)
        finally:
            m.kl_batch_destroy(b)
