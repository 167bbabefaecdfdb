"""Which kernel the linear surrogate's inputs go to (paper_2601_07891_amd/csrc/score_linear_rule.h): at sizes
where both sides were timed, to the faster one.  CPU only."""
import pytest

from tests import deal


@pytest.mark.parametrize("rows,Dh,H,form", [
    (1024, 4096, 8, "rows"), (4641, 4096, 8, "rows"), (6106, 4096, 8, "rows"), (5471, 5120, 8, "rows"),
    (5536, 3072, 8, "rows"), (7449, 2048, 8, "rows"),                        # rounds that the stream does not beat
    (6838, 4096, 8, "stream"), (6253, 5120, 8, "stream"), (6187, 3072, 8, "stream"), (8303, 2048, 8, "stream"),
    (14895, 1024, 8, "narrow"), (13674, 2048, 8, "narrow"), (13674, 3072, 4, "narrow"), (29788, 512, 8, "narrow"),
    (11233, 2048, 1, "narrow"), (62503, 512, 2, "narrow"),
    (12210, 2048, 8, "stream"), (16279, 3072, 8, "stream"), (16384, 1024, 8, "narrow"), (16604, 1024, 8, "stream"), (16384, 4096, 8, "stream"), (70315, 512, 1, "stream"),
    (6145, 2560, 2, "stream"), (7449, 2048, 2, "short"), (59573, 256, 8, "narrow"), (120000, 128, 8, "stream"),
    (262144, 5120, 8, "stream"), (4113, 4096, 16, "stream"), (4096, 4096, 16, "short"),
    (20000, 5120, 15, "narrow"), (70000, 5120, 15, "wide"),                  # W leaves the stream no room
])
def test_inputs_go_to_the_faster_kernel(rows, Dh, H, form):
    assert deal.linear_form(rows, Dh, H) == form


def test_the_benchmark_names_the_kernels_that_run():
    import random

    import bench
    rng = random.Random(3)
    names = {"rows": "score_linear_rows_kernel", "stream": "score_linear_stream_kernel",
             "short": "score_linear_short_kernel"}
    for _ in range(150):
        Dh, H = 64 * rng.randint(1, 120), rng.choice([1, 2, 3, 4, 8, 8, 12, 16])
        rows = int(2 ** rng.uniform(0, 19))
        if H * (Dh * 2 + 64) <= 160 * 1024:
            form = deal.linear_form(rows, Dh, H)
            assert bench.linear_kernel(rows, Dh, H) == names.get(form, "score_linear_kernel"), (rows, Dh, H, form)
        heads, group, bound, window = rng.randint(1, 600), rng.randint(1, 16), int(2 ** rng.uniform(0, 17)), rng.choice([0, 40, 128])
        kind = deal.form(heads, group, bound, window, bound).split()[0]
        assert bench.attend_kernel(heads, group, bound, window) == ("attend_list_kernel" if kind in ("list", "block")
                                                                     else "attend_split_kernel"), (heads, group, bound, window)
