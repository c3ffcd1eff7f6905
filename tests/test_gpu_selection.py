"""Which configuration an unrecorded problem size runs: one that takes its rows."""
import json
import os

import pytest
import torch

pytestmark = pytest.mark.gpu

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SECOND = ("advec_u", "diff_uvw", "advec_diff", "step")
LES = ("advec_u_2i5", "diff_smag")


@pytest.fixture()
def m():
    from paper_2303_12374_amd import kl
    yield kl
    kl.kl_set_wisdom_dir(None)


def kernel_id(m, name):
    return next(k for k, n in m.KERNEL_NAMES.items() if n == name)


def selected(m, kernel, dtype, size):
    """Name of the configuration selected for a padded grid, and whether it takes the grid."""
    gc = 3 if kernel in LES else 1
    g = m.Grid(*size, dtype=dtype, gc=gc)
    k = kernel_id(m, kernel)
    i = m.kl_selected_variant(g, k)
    return m.kl_variant_name(k, dtype, i), m.kl_variant_eligible(g, k, i, [None] * 7)


def write(m, path, recs):
    """Wisdom of this GPU: {kernel: [(dtype, size, configuration)]}."""
    p = torch.cuda.get_device_properties(0)
    for kernel, rows in recs.items():
        (path / (kernel + ".wisdom")).write_text("".join(json.dumps(
            {"kernel": kernel, "dtype": "f32" if dt == 0 else "f64", "problem_size": list(s), "variant": v,
             "device": p.name, "arch": p.gcnArchName.split(":")[0], "time_ms": 1.0}) + "\n" for dt, s, v in rows))
    m.kl_set_wisdom_dir(str(path))


# rows longer than any row-flattened tile takes, next to records that name one;
# rows of fewer points than the paper's schemes' tile takes
@pytest.mark.parametrize("size", [(768, 300, 100), (560, 300, 100), (640, 232, 202), (704, 400, 80), (516, 130, 130),
                                  (224, 534, 345), (1028, 200, 64), (4, 256, 256), (1, 512, 512), (5, 30, 20),
                                  (600, 40, 20), (1000, 16, 16), (2048, 4, 64)], ids=lambda s: "x".join(map(str, s)))
@pytest.mark.parametrize("dtype", [0, 1], ids=["f32", "f64"])
def test_selected_configuration_takes_the_grid(m, dtype, size):
    m.kl_set_wisdom_dir(os.path.join(ROOT, "wisdom"))
    for kernel in SECOND + LES:
        name, ok = selected(m, kernel, dtype, size)
        assert ok, (kernel, name)


def test_unusable_nearest_record_is_passed_over(m, tmp_path):
    """FP64 rows of 768 points are 384 chunks; the nearest record's tile takes 256."""
    write(m, tmp_path, {"step": [(1, (768, 700, 100), "step_v2_b64x4_k32_x2_nt1_w1_h3"), (1, (760, 300, 100), "rf_t512")]})
    assert selected(m, "step", 1, (768, 300, 100))[0] not in ("rf_t512", m.kl_variant_name(m.STEP, 1, 0))
