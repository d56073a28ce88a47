"""Which tensors the no-allocation report accepts: the size rule its callers
plan with (r and u of m, c and v of n, column partial sums, error, fold and
statistics partials, in doubles), whatever form of the report runs."""
import random

from paper_2609_30342_amd import rikfad as R


def _planned_words(m, n):
    ncb, stripe = -(-n // 256), 1024
    while stripe > 16 and ncb * -(-m // stripe) < 2048:
        stripe >>= 1
    while -(-m // stripe) > 65535:
        stripe <<= 1
    parts = -(-m // 256) if n <= 1024 else -(-m // stripe)
    return (2 * (m + n) + parts * n + 2 * -(-m // 16) + 4 * -(-n // 4)
            + 2 * -(-max(m, n) // 4096) + 6)


def test_noalloc_accepts_what_fits_the_planned_size():
    limit = R.rikfad_friction_report_noalloc_max_bytes()
    rng = random.Random(1)
    for _ in range(4000):
        m, n = (int(2 ** rng.uniform(0, 20.9)) for _ in range(2))
        got, plan = R.rikfad_friction_report_workspace_bytes(m, n), 8 * _planned_words(m, n)
        assert got >= plan, (m, n)
        assert (got <= limit) == (plan <= limit), (m, n, got, plan)
