"""The lines between light and heavy rows that a batch's plans are made with (executor.plan_limits)."""
import pytest
import torch

from paper_2106_05609_amd.executor import _windowed, plan_limits


@pytest.mark.parametrize("rows,entries,longest,want", [
    (0, 0, 0, None),
    (3_750, 89_108, 269, (64, 32)),                      # few entries: a launch waits for its longest row
    (25_000, 462_196, 141, None),                        # hardly longer than the line
    (15_000, 642_765, 563, (86, 64)),                    # twice the mean
    (50_000, 1_826_185, 1_705, (74, 64)),
    (100_000, 4_311_623, 3_302, (128, 64)),
    (116_664, 1_979_499, 290, None),                     # a short walk beside the launch
    (600_000, 50_318_351, 17_482, (256, 128)),
    (312_500, 6_869_018, 3_825, (512, 256)),             # many rows hide a long one's walk: the plan's own limits
    (262_144, 3_000_000, 2_000, (512, 256)),
    (262_143, 3_000_000, 2_000, (256, 128)),
    (131_072, 9_999_999, 2_000, (256, 128)),
    (131_071, 3_000_000, 2_000, (128, 64)),
    (300_000, 2_999_999, 2_000, (64, 64)),
    (300_000, 10_000_000, 2_000, (256, 128)),
    (4_000, 480_381, 152, None),                         # long rows of like lengths
    (1_000, 600_000, 5_000, (512, 64)),                  # no line above 512
    (1, 513, 513, (512, 32)),
])
def test_lines_follow_the_batch(rows, entries, longest, want):
    got = plan_limits(rows, entries, longest)
    assert got == (None if want is None else dict(heavy_threshold=want[0], chunk=want[1]))


def test_rows_above_512_are_always_cut():
    for rows in (1, 100, 10_000, 1_000_000):
        for mean in (1, 30, 400, 2_000):
            got = plan_limits(rows, rows * mean, max(513, mean))
            assert got is not None and got["heavy_threshold"] <= 512 and got["chunk"] <= 128


@pytest.mark.parametrize("max_F,rows", [(256, 16384), (1433, 16384), (184, 22795), (64, 65536), (1, 1 << 20)])
def test_windows_of_short_chunks(max_F, rows):
    assert _windowed(None, max_F) is None
    assert _windowed(dict(heavy_threshold=512, chunk=256), max_F) == dict(heavy_threshold=512, chunk=256)
    assert _windowed(dict(heavy_threshold=256, chunk=128), max_F) == dict(heavy_threshold=256, chunk=128, window_rows=rows)


@pytest.mark.parametrize("given", [None, {}, dict(xcd_ranges=2)])
def test_options_of_a_batch_are_all_or_none(given, monkeypatch):
    """A caller's options reach each of the batch's plans as they are, an empty dict too; without any the limits do."""
    from paper_2106_05609_amd import executor
    nb, nv = 3, 5
    rowptr = torch.tensor([0, 600, 601, 602], dtype=torch.int32)             # columns 0 and 4 of 300 and 301 entries
    col = torch.cat([torch.zeros(300), torch.full((300,), 4), torch.tensor([1, 4])]).int()
    colptr, row = torch.tensor([0, 300, 301, 301, 301, 602], dtype=torch.int32), torch.zeros(602, dtype=torch.int32)
    seen = []
    monkeypatch.setattr(executor.B, "gas_plan_create", lambda *a, options=None, **k: seen.append(options))
    bg = executor.BatchGraph(nb, torch.arange(nv).int(), rowptr, col, None, colptr, row, max_F=256, normalise=False, plan_options=given)
    bg.plan_t_all
    limits = [_windowed(plan_limits(*p), 256) for p in ((3, 602, 600), (3, 301, 300), (5, 602, 301))]
    assert limits[0] is not None
    assert seen == (limits if given is None else [given] * 3)
