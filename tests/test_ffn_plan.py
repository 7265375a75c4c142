"""How the products of the expert networks are laid out, asked from the library on the host (no GPU)."""
import pytest

import gpu_helpers as H
from paper_2406_00023_amd import binding as B
from paper_2406_00023_amd import inputs as I


def _cfg(T, E, d, Hh, C, k=2, mode=I.MODE_BIDIR):
    return B.make_config(I.EtrShape("p", 1, T=T, d=d, E=E, D=8, k=k, capacity=C, H=Hh, dtype=I.DT_BF16, mode=mode, recipe="iso"))


@pytest.mark.parametrize("T,E,d,Hh", [(32, 16, 2048, 5632), (256, 32, 4096, 2816), (500, 64, 512, 1024)])
@pytest.mark.parametrize("product", [0, 1])
def test_capacity_above_the_batch_adds_no_workgroups(T, E, d, Hh, product):
    """A buffer made once for the largest batch: the few-rows grid follows the rows that the batch can fill."""
    tight = H.ffn_plan(_cfg(T, E, d, Hh, T), product)
    assert tight[0] == H.ROWS
    for C in (16 * T, 4096, 65536):
        kernel, groups = H.ffn_plan(_cfg(T, E, d, Hh, C), product)
        assert kernel == H.ROWS
        assert groups <= 1.2 * tight[1] + 8, (C, groups, tight)      # (one more partial row tile than with C = T)


def test_few_rows_launch_is_within_what_one_launch_may_hold():
    """2^32 threads: an expert count, a capacity and a width that the config check accepts must not pass it."""
    for product in (0, 1):
        kernel, groups = H.ffn_plan(_cfg(1000, 64, 1024, 4096, 131072), product)
        assert kernel == H.ROWS
        assert groups * 256 < 2 ** 32, (product, groups)
