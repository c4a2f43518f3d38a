"""The bench's FP64 roofline entry names kernels that exist and prices the operations made."""
import os
import re

import pytest

import bench

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_1507_00895_amd", "csrc")


class _Lib:
    def df_ladder_variant(self, n_nu, prec):
        return "gjb_o3" if n_nu <= 64 else "gjb"


@pytest.mark.parametrize("n_nu", [16, 48, 50, 64, 80, 96, 128])
def test_kernels_exist_and_the_fraction_is_one(n_nu):
    src = "".join(open(os.path.join(CSRC, f)).read() for f in sorted(os.listdir(CSRC))
                  if f.endswith((".hip", ".hpp")))
    r = bench.as_run(bench.roofline_of(0, _Lib(), 31, 1024, n_nu, 10.0), n_nu)
    for name in r["launches"]:
        assert re.search(r"\b" + name.split("<")[0] + r"\(LadderArgs", src), name
    assert r["kernel"] == r["launches"][1]
    # fewer operations than the dense inverse, and the fraction follows them
    assert r["executed_flops_per_launch"] < r["algorithmic_flops_per_launch"] * 1.6
    assert r["frac"] == pytest.approx(r["executed_flops_per_launch"] / 10e-3 / 1e12 / 78.6)


def test_product_counts():
    assert [bench.sym_products(n) for n in (4, 6, 8)] == [32, 100, 224]
