"""kl_euler on rows around 256 chunks of 16 bytes (several rows a block below, one
above) and 512 (several blocks a row above)."""
import numpy as np
import pytest
import torch

from paper_2303_12374_amd import inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("layout", ["padded", "plain"])
@pytest.mark.parametrize("gc", [1, 3])
@pytest.mark.parametrize("bc", [0, 1, 2], ids=["zerograd", "nopen", "zperiodic"])
@pytest.mark.parametrize("dtype,itot", [(0, 1023), (0, 1024), (0, 1025), (0, 2047), (0, 2048), (0, 2052), (0, 4099),
                                        (1, 511), (1, 512), (1, 513), (1, 560), (1, 1024), (1, 1026), (1, 2049)])
def test_long_rows_advance_like_short_ones(dtype, itot, bc, gc, layout):
    """Bitwise the update of the same values with x and y exchanged (short rows): the
    update is pointwise, and every ghost layer is the ghost fill's."""
    from paper_2303_12374_amd import kl as m
    jtot, ktot = 7, 4
    rng = np.random.RandomState(7)
    v = [rng.uniform(-1, 1, (ktot, jtot, itot)) for _ in range(6)]
    out = []
    for swap in (False, True):
        size = (jtot, itot, ktot) if swap else (itot, jtot, ktot)
        g = m.Grid(*size, dtype=dtype, bc=bc, gc=gc, layout=inputs.plain_layout(*size, gh=gc) if layout == "plain" else None)
        x = [g.upload(np.ascontiguousarray(a.transpose(0, 2, 1)) if swap else a) for a in v]
        m.kl_fill_ghosts(g, *x[:3])
        m.kl_euler(g, 0.37, *x)
        chk = [t.clone() for t in x[:3]]
        m.kl_fill_ghosts(g, *chk)
        for a, b in zip(x[:3], chk):
            assert torch.equal(torch.nan_to_num(a, nan=77.0), torch.nan_to_num(b, nan=77.0))
        out.append([g.interior(t).cpu().numpy() for t in x[:3]])
    for a, b in zip(*out):
        assert np.array_equal(a, b.transpose(0, 2, 1))


def test_long_rows_take_no_longer_than_short_ones():
    """The same points in rows of 2048 and of 256 (FP64): with one block per row
    the long ones took 1.5 times as long."""
    from paper_2303_12374_amd import kl as m

    def best(size):
        g = m.Grid(*size, dtype=1)
        x = [g.full(0.5) for _ in range(6)]
        e = [torch.cuda.Event(True) for _ in range(2)]
        ts = []
        for _ in range(12):
            e[0].record()
            for _ in range(50):
                m.kl_euler(g, 1e-9, *x)
            e[1].record()
            torch.cuda.synchronize()
            ts.append(e[0].elapsed_time(e[1]))
        return min(ts)

    assert best((2048, 16, 128)) < 1.25 * best((256, 128, 128))
