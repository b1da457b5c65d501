"""The number of segments that the workspace of the bf16 forward's linear branch has room for where the call chooses, read off the size
that a call reports (three states per segment and output head), on both sides of every line of the rule.  It is the most that a call
takes: how many it does take, or whether it runs in one pass instead, is test_scan_form.py's."""
import pytest

from paper_2602_03681_amd import binding as nb


def segments(H, L, d, **kw):
    size = lambda n: nb.fwd_workspace_bytes(nb.make_fwd_params(1, H, L, d, 64, nb.NATS_BF16, gdn_segments=n, **kw))
    more, rest = divmod(size(0) - size(1), 3 * H * kw.get("group", 1) * d * d * 4)
    assert rest == 0
    return 1 + more


@pytest.mark.parametrize("H,chunks,n", [
    (1, 1, 1), (1, 15, 1), (1, 16, 4), (1, 19, 4), (1, 20, 5),   # none below 16 chunks, then 4 chunks a segment ...
    (1, 64, 16), (1, 68, 16), (1, 128, 22), (1, 256, 32),        # ... until n^2 is over 4 chunks
    (4, 128, 22), (8, 64, 16),
    (85, 64, 3), (86, 64, 1), (128, 64, 1), (256, 64, 1),        # no more blocks than fill the chip, and never two segments
])
@pytest.mark.parametrize("d", [64, 128])
def test_rule(H, chunks, n, d):
    assert segments(H, 64 * chunks, d) == n


def test_groups_count_output_heads():
    assert segments(43, 4096, 64, group=2) == segments(86, 4096, 64) == 1
    assert segments(42, 4096, 64, group=2) == segments(84, 4096, 64) == 3
