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


@pytest.mark.parametrize("product,E,rows,d,Hh,kernel", [
    # the kernel measured fastest by a quarter or more (us of the others in the comment)
    (0, 16, 8, 2048, 5632, "ROWS"),                # 120; 256-row tiles 165
    (0, 8, 160, 1536, 640, "ROWS"),                # 19; 38
    (0, 32, 96, 4096, 128, "ROWS"),                # 22; 85
    (1, 4, 256, 1080, 2744, "ROWS"),               # 26; register-staged 45, 256-row tiles 65
    (0, 32, 512, 768, 384, "PERSISTENT"),          # 27; few rows 56
    (0, 8, 450, 640, 11008, "PERSISTENT"),         # 126; 332
    (1, 16, 160, 2232, 1472, "PERSISTENT"),        # 43; 57
    (1, 64, 384, 1024, 2816, "PERSISTENT"),        # 159; 373
    (0, 8, 192, 1080, 2744, "PERSISTENT_TAIL"),    # 35; 48 and register-staged 47
    (0, 16, 1024, 520, 1000, "PERSISTENT_TAIL"),   # 42; 107 and 63
    (0, 32, 1024, 64, 2048, "RING"),               # 72; few rows 219
    (1, 64, 1024, 1024, 64, "RING"),               # 56; 132
    (0, 4, 256, 1080, 2744, "STAGED"),             # 27; few rows 36, 256-row tiles 36
    (0, 16, 256, 520, 1000, "STAGED"),             # 18; 31 and 26
])
def test_kernel_choice_at_measured_points(product, E, rows, d, Hh, kernel):
    cfg = _cfg(rows * E, E, d, Hh, rows, k=1)
    assert H.ffn_plan(cfg, product, gathered=False)[0] == getattr(H, kernel)
