"""Which kernel a pooled lookup takes: the library's choice, on the host."""
from paper_2512_05831_amd import eb
from route_util import PLAIN, TEAM, WAVE, route


def test_hinted_rows_no_16_byte_chunk_divides_are_cached():
    """Such rows share cache lines, and a batch may name them again: the hint
    moves neither their loads past the caches nor, where tables that do not fit
    the L2s are reused, eight tables' rows into the caches at a time.  Only
    where tables far beyond the caches see hardly a row twice are they streamed."""
    for D, dtype in ((227, eb.EB_F32), (217, eb.EB_F32), (257, eb.EB_F16), (236, eb.EB_BF16)):
        r = route(D, dtype, 9, 10272, 47, 720_000, hint=True)
        assert (r.kernel, r.non_temporal, r.xcd_runs) == (WAVE, 0, 0), D
        r = route(D, dtype, 38, 7880, 14, 11_000, hint=True)
        assert (r.kernel, r.non_temporal, r.xcd_runs) == (WAVE, 0, 1), D
        for rows, nt in ((2_000_000, 0), (4_000_000, 1)):  # a row in 6 used, in 12
            r = route(D, dtype, 4, 34679, 10, rows, hint=True)
            assert (r.kernel, r.non_temporal, r.xcd_runs) == (WAVE, nt, 1), (D, rows)
    r = route(128, eb.EB_F32, 8, 2048, 40, 1_000_000, hint=True)  # whole 16-byte chunks: streamed, by teams
    assert (r.kernel, r.non_temporal, r.xcd_runs) == (TEAM, 1, 1)


def test_large_batches_take_the_wave_kernel_where_a_team_is_a_wave_too():
    """Bags that teams narrower than a wave would take go to the wave kernel
    from four passes, by the ids a row block gathers and not by those its bags
    name; up to 8192 bags from two, gathered or not."""
    for D, dtype, four, full in ((64, eb.EB_F32, 16, 24), (128, eb.EB_F32, 8, 12), (256, eb.EB_BF16, 8, 12),
                                 (256, eb.EB_F32, 4, 6)):
        assert route(D, dtype, 2, 55087, four - 1, 1_000_000).kernel == TEAM
        assert route(D, dtype, 2, 55087, four, 1_000_000).kernel == WAVE
        assert route(D, dtype, 2, 55087, full - 1, 1_000_000, local=125_000).kernel == TEAM
        assert route(D, dtype, 2, 55087, full, 1_000_000, local=125_000).kernel == WAVE
        assert route(D, dtype, 2, 55087, full, 1_000_000, hint=True).kernel == TEAM
        assert route(D, dtype, 2, 4000, 1, 1_000_000, hint=True).kernel == WAVE
    for D, dtype, four in ((64, eb.EB_F16, 32), (32, eb.EB_F32, 32), (16, eb.EB_F32, 64), (8, eb.EB_F16, 64)):
        assert route(D, dtype, 2, 55087, four - 1, 1_000_000).kernel == TEAM
        assert route(D, dtype, 2, 55087, four, 1_000_000).kernel == WAVE
        assert route(D, dtype, 2, 55087, 4 * four - 1, 1_000_000, local=250_000).kernel == TEAM
        assert route(D, dtype, 2, 55087, 4 * four, 1_000_000, local=250_000).kernel == WAVE
        assert route(D, dtype, 4, 40000, four, 1_000_000).kernel == (TEAM if four < 64 else WAVE)  # five there
        assert route(D, dtype, 4, 40000, min(64, four * 5 // 4), 1_000_000).kernel == WAVE
    assert route(64, eb.EB_F16, 2, 4000, 16, 1_000_000, local=250_000).kernel == WAVE
    assert route(64, eb.EB_F16, 2, 4000, 15, 1_000_000).kernel == TEAM
    assert route(64, eb.EB_F16, 2, 55087, 100, 0).kernel == TEAM  # no rows at all


def test_small_batches_are_cached_unless_no_row_comes_back():
    for D, dtype in ((128, eb.EB_F32), (64, eb.EB_F16), (189, eb.EB_F16)):
        for bags in (300, 2000):
            for rows, nt in ((20_000, 0), (5_000_000, 1)):
                r = route(D, dtype, 4, bags, 49, rows, hint=True)
                assert (r.kernel, r.non_temporal) == (WAVE, nt), (D, bags, rows)
                assert route(D, dtype, 4, bags, 49, rows).non_temporal == 0
    assert route(128, eb.EB_F32, 4, 300, 49, 20_000, hint=True, align=2).kernel == PLAIN  # fp32 rows off 4 bytes


def test_bags_of_one_id_run_in_order_on_each_xcd():
    for D, dtype in ((36, eb.EB_BF16), (128, eb.EB_F32), (267, eb.EB_F16)):
        assert not route(D, dtype, 1, 128, 1, 1_000_000).xcd_runs
        for bags in (129, 2000, 50000):
            for hint in (False, True):
                r = route(D, dtype, 1, bags, 1, 1_000_000, hint=hint)
                assert r.kernel == TEAM or r.xcd_runs
                r = route(D, dtype, 1, bags, 2, 1_000_000)
                assert not r.xcd_runs
