"""Sizes of the friction report's workspace: at least what the form that runs
lays out (counted here from its buffers), and within the static scratch for
exactly the tensors that the size rule callers plan with puts there."""
import random

import pytest

from paper_2609_30342_amd import rikfad as R


def _stripes(m, n):
    ncb, stripe = -(-n // 256), 1024
    while stripe > 16 and ncb * -(-m // stripe) < 2048:
        stripe >>= 1
    while -(-m // stripe) > 65535:
        stripe <<= 1
    return -(-m // stripe)


def _planned_words(m, n):
    """The rule: r and u of m, c and v of n, column partial sums, error, fold
    and statistics partials and six results, in doubles."""
    parts = -(-m // 256) if n <= 1024 else _stripes(m, n)
    return (2 * (m + n) + parts * n + 2 * -(-m // 16) + 4 * -(-n // 4)
            + 2 * -(-max(m, n) // 4096) + 6)


def _laid_out_words(m, n):
    """What the form that runs writes.  One pass over xi (n <= 16384): C and v
    padded to whole groups of 4, a row of column partial sums and a pair of
    errors and of norms per workgroup (at least 16 rows each up to 1024
    columns, at most 256 of them), a pair per 16 columns of either fold, the
    results.  Two passes: one row of column partial sums per stripe, a pair
    per 16 rows of errors and per 4096 elements of the vector statistics."""
    fold = 4 * -(-n // 16) + 6
    if n <= 1024:
        nblk = -(-m // max(16, -(-m // 256)))
        return 2 * (-n % 4 + n) + nblk * (-n % 4 + n + 4) + fold
    return 2 * (m + n) + _stripes(m, n) * n + 2 * -(-m // 16) + fold + 2 * -(-max(m, n) // 4096)


@pytest.mark.parametrize("n", [1, 2, 3, 4, 5, 255, 1024, 16385, 50257])
def test_workspace_holds_what_its_form_writes(n):
    for m in [1, 2, 15, 16, 17, 31, 33, 255, 256, 257, 1000, 1025, 4099, 5000, 32767, 32769, 50257,
              70000, 131073, 200000, 524287, 524289, 980000, 2000003]:
        got = R.rikfad_friction_report_workspace_bytes(m, n)
        assert got >= 8 * _laid_out_words(m, n), (m, n, got)


def test_noalloc_accepts_what_fits_the_planned_size():
    limit = R.rikfad_friction_report_noalloc_max_bytes()
    rng = random.Random(1)
    sizes = [tuple(int(2 ** rng.uniform(0, 20.9)) for _ in range(2)) for _ in range(4000)]
    for n in (1, 2, 3, 4):                  # both sides of the limit
        edge = next(m for m in range(1 << 20, 0, -1) if 8 * _planned_words(m, n) <= limit)
        sizes += [(edge + d, n) for d in range(-40, 41)]
    for m, n in sizes:
        got, plan = R.rikfad_friction_report_workspace_bytes(m, n), 8 * _planned_words(m, n)
        assert got >= plan, (m, n)
        assert (got <= limit) == (plan <= limit), (m, n, got, plan)
