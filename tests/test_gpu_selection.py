"""Which configuration an unrecorded problem size runs: one that takes its rows,
the record of nearly the same size where there is one, and no record of a
size far away; and all configurations that the rules can name exist."""
import json
import os
import re

import pytest
import torch

from paper_2303_12374_amd import inputs

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


@pytest.mark.parametrize("kernel,dtype,name", [("diff_uvw", 0, "zl3_v4_b64x8_k256_x3_nt1"),
                                               ("advec_diff", 1, "ad_v2_b64x4_k64_x2_nt1"),
                                               ("step", 0, "step_v4_b64x8_k64_x2_nt1_w1_h3y")])
def test_record_of_nearly_the_same_size_decides(m, tmp_path, kernel, dtype, name):
    write(m, tmp_path, {kernel: [(dtype, (256, 256, 256), name), (dtype, (248, 256, 250), "default")]})
    assert selected(m, kernel, dtype, (256, 254, 256))[0] == name  # 0.8%
    assert selected(m, kernel, dtype, (256, 192, 256))[0] != name  # a quarter off


@pytest.mark.parametrize("kernel", ["advec_u", "diff_uvw"])
@pytest.mark.parametrize("dtype", [0, 1], ids=["f32", "f64"])
def test_small_grid_does_not_take_a_far_records_tile(m, tmp_path, kernel, dtype):
    """500x20x30: a march of 32 levels on one tile column leaves the chip idle."""
    v = 4 if dtype == 0 else 2
    far = f"zl_v{v}_b64x8_k32_x2_nt1_w1"
    write(m, tmp_path, {kernel: [(dtype, (512, 128, 128), far)]})
    assert selected(m, kernel, dtype, (500, 20, 30))[0] != far


@pytest.mark.parametrize("kernel,dtype,size,name", [
    ("step", 1, (264, 100, 60), "rf_t512"), ("step", 0, (532, 64, 64), "rf_t512"), ("step", 0, (510, 300, 100), "rf_t512"),
    ("step", 1, (614, 10, 112), "step_v2_b64x4_k8_x0_nt0"), ("step", 0, (1302, 60, 60), "step_v1_b64x4_k8_x0_nt0"),
    ("diff_uvw", 1, (614, 10, 112), "zl_v2_b64x8_k8_x0_nt0_w1"), ("diff_uvw", 0, (1136, 12, 137), "default"),
    ("advec_diff", 0, (1239, 91, 91), "default"), ("advec_diff", 0, (1136, 23, 267), "ad_v4_b64x4_k8_x0_nt0"),
    ("advec_u", 0, (520, 100, 60), "zc_v2_b64x1_k16_x1"), ("advec_u", 0, (501, 100, 50), "zc_v1_b64x1_k16_x1"),
    ("advec_u", 1, (178, 166, 18), "rf_t512"), ("advec_u", 1, (336, 200, 120), "rf_t512")])
def test_small_grids_of_long_rows(m, tmp_path, kernel, dtype, size, name):
    """Short marches where few points have to fill the chip, whatever the records far away say."""
    v = 4 if dtype == 0 else 2
    far = {"step": f"step_v{v}_b64x8_k64_x2_nt1_w1_h3y", "advec_diff": f"ad_v{v}_b64x4_k64_x2_nt1"}
    write(m, tmp_path, {kernel: [(dtype, (512, 512, 512), far.get(kernel, f"zl_v{v}_b64x8_k32_x2_nt1_w1"))]})
    got, ok = selected(m, kernel, dtype, size)
    assert ok and got == name


def test_every_configuration_the_rules_name_exists(m):
    """A misspelt name would quietly fall to the nearest record."""
    src = open(os.path.join(ROOT, "paper_2303_12374_amd", "csrc", "api.cpp")).read()
    rule = src[src.index("const char *wide_rows_tile"):src.index("int select_variant")]
    names = set(re.findall(r'"((?:zc|zl|ad|step|a5|s2|rf)_[a-z0-9_]+)"', rule))
    assert len(names) >= 12
    known = {m.kl_variant_name(k, d, i) for k in range(6) for d in (0, 1) for i in range(m.kl_num_variants(k, d))}
    assert names <= known


def test_selection_follows_the_rows_not_the_layout(m):
    """The choice is by size; a layout that it does not fit is handled at the call."""
    m.kl_set_wisdom_dir(os.path.join(ROOT, "wisdom"))
    for size in ((300, 40, 40), (64, 64, 64), (516, 130, 130)):
        for kernel in SECOND:
            k = kernel_id(m, kernel)
            a = m.kl_selected_variant(m.Grid(*size, dtype=1), k)
            m.kl_clear_plan_cache()
            assert a == m.kl_selected_variant(m.Grid(*size, dtype=1, layout=inputs.plain_layout(*size)), k)
