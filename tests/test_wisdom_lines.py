"""Which lines of a wisdom file count: the reader parses only those that can hold
the field type, so spellings of it, other types and unknown names are tried."""
import json

import pytest

from paper_2303_12374_amd import kl

REC = {"kernel": "advec_u", "dtype": "f32", "problem_size": [64, 64, 64], "device": "A", "arch": "gfx950"}


def lookup(tmp_path, lines, dtype=0, size=(64, 64, 64)):
    (tmp_path / "advec_u.wisdom").write_text("\n".join(lines) + "\n")
    return kl.kl_wisdom_lookup(str(tmp_path), kl.ADVEC_U, dtype, "A", "gfx950", *size)


def line(n, dtype="f32", **more):
    return json.dumps({**REC, "dtype": dtype, "variant": kl.kl_variant_name(kl.ADVEC_U, 0, n), **more})


@pytest.mark.parametrize("spelt", ['"dtype":"f32"', '"dtype" :  "f32"', '"dtype": "f3\\2"', '"dtype": "\\f32"'])
def test_spellings_of_the_type(tmp_path, spelt):
    text = line(3).replace('"dtype": "f32"', spelt)
    want = (kl.kl_variant_name(kl.ADVEC_U, 0, 3), 1) if "\\f" not in spelt else ("default", 5)
    assert lookup(tmp_path, [text]) == want


def test_other_type_does_not_count_although_it_names_this_one(tmp_path):
    assert lookup(tmp_path, [line(3, "f64", note="f32")]) == ("default", 5)
    assert lookup(tmp_path, [line(3, "f64", note="f32"), line(4)])[0] == kl.kl_variant_name(kl.ADVEC_U, 0, 4)


def test_unknown_name_and_broken_lines_are_passed_over(tmp_path):
    good = line(5)
    bad = [line(3, variant="zl_v4_b64x8_k7"), good[:-1], good + "}", good.replace("64, 64", "64"), '"f32"', "f32"]
    assert lookup(tmp_path, [good] + bad) == (kl.kl_variant_name(kl.ADVEC_U, 0, 5), 1)
    assert lookup(tmp_path, bad) == ("default", 5)


def test_every_name_of_a_registry_is_found(tmp_path):
    for dtype, spelt in ((0, "f32"), (1, "f64")):
        for n in range(kl.kl_num_variants(kl.ADVEC_U, dtype)):
            name = kl.kl_variant_name(kl.ADVEC_U, dtype, n)
            assert lookup(tmp_path, [line(0, spelt, variant=name)], dtype) == (name, 1)


def test_long_strings_and_numbers(tmp_path):
    more = {"note": "x" * 5000, "time_ms": 1.2345678901234567e-3, "big": 10 ** 50, "nest": {"a": [1, [2, "]}"]]}}
    assert lookup(tmp_path, [line(3, **more)], size=(65, 64, 64)) == (kl.kl_variant_name(kl.ADVEC_U, 0, 3), 2)
