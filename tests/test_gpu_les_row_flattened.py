"""Row-flattened configurations of advec_u_2i5 and diff_smag (rf_t512) where
they can go wrong: the shortest rows, partial last chunks, one and several
segments per row (line-aligned, equal, rounded up), row blocks with a
remainder, one and two levels per tile, misaligned rows, all boundary modes,
one and three ghost cells; and a grid above the size from which tendencies are
streamed.  Each is compared bitwise, ghost and padding cells included, with
the default configuration, which the oracle tests hold."""
import pytest
import torch

from paper_2303_12374_amd import inputs

pytestmark = pytest.mark.gpu

SHAPES = [(8, 3, 2), (9, 1, 3), (33, 40, 4), (255, 13, 5), (256, 19, 3), (301, 23, 7), (390, 17, 3), (516, 9, 4),
          (700, 11, 2), (1023, 5, 3)]


def compare(m, g, dtype):
    f = [g.full(0.25) for _ in range(3)]
    m.kl_generate_fields(g, 57, *f)
    m.kl_fill_ghosts(g, *f)
    evisc = f[0].abs() + 0.125
    m.kl_fill_scalar(g, evisc)
    for kernel, nout in ((m.ADVEC_U_2I5, 1), (m.DIFF_SMAG, 3)):
        if kernel == m.ADVEC_U_2I5 and g.gc < 3:
            continue
        names = [m.kl_variant_name(kernel, dtype, i) for i in range(m.kl_num_variants(kernel, dtype))]
        res = []
        for i in (0, names.index("rf_t512")):
            out = [g.full(-5.0) for _ in range(3)]
            for n, x in enumerate(out):
                g.interior(x).fill_(0.5 + n)
            fields = f + out + ([evisc] if kernel == m.DIFF_SMAG else [])
            assert m.kl_variant_eligible(g, kernel, i, fields)
            m.kl_launch_variant(g, kernel, i, fields)
            res.append(out)
        for a, b in zip(*res):
            assert torch.equal(a, b), names
        assert not torch.equal(res[0][0], g.full(-5.0))


@pytest.mark.parametrize("layout", ["padded", "plain"])
@pytest.mark.parametrize("bc", [0, 1, 2], ids=["zerograd", "nopen", "zperiodic"])
@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: "x".join(map(str, s)))
@pytest.mark.parametrize("dtype", [0, 1], ids=["f32", "f64"])
def test_les_row_flattened_bitwise_equals_default(dtype, shape, bc, layout):
    from paper_2303_12374_amd import kl as m
    for gc in (1, 3):
        lay = inputs.plain_layout(*shape, gh=gc) if layout == "plain" else None
        compare(m, m.Grid(*shape, dtype=dtype, bc=bc, gc=gc, layout=lay), dtype)


@pytest.mark.parametrize("dtype", [0, 1], ids=["f32", "f64"])
def test_les_row_flattened_streams_large_tendencies(dtype):
    from paper_2303_12374_amd import kl as m
    g = m.Grid(301, 256, 211, dtype=dtype, gc=3)
    assert 4 * (8 if dtype else 4) * g.npoints > 256e6
    compare(m, g, dtype)
