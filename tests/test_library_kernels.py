"""The built library holds no kernel that its dispatch cannot reach: two columns per thread in the
register-tiled hop kernel (k_hop<..., CT, MODE, ...>) are taken by BF16 blocks only; FP64 and FP32
blocks of three columns and more always go to the LDS-staged kernels."""

import os
import re

import pytest

LIB = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_0907_3261_amd", "libwdsolve.so")


def test_pairs_of_columns_exist_for_bf16_only():
    if not os.path.exists(LIB):
        pytest.skip("the library is not built")
    with open(LIB, "rb") as f:
        names = set(re.findall(rb"k_hopINS_\d(St\w+?)E(?:\w*?)Li(\d)ELi(\d)ELi\d", f.read()))
    pairs = {n[0] for n in names if n[1] == b"2"}
    assert pairs == {b"StBF16"}, sorted(names)
