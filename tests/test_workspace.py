"""Workspace sizes that the library asks for (host arithmetic, no GPU)."""
import pytest


@pytest.mark.parametrize("t", [0, 1])
@pytest.mark.parametrize("q", [0, 1, 2])
def test_compress_asks_for_what_it_uses(q, t):
    """Per 1024-value chunk an outlier count, a width word and a record size
    of 4 bytes each and 16 flags of 64 lanes; nothing by the value's size,
    since the outliers go straight to the packed stream."""
    import paper_2407_15037_amd as lcq
    L = lcq.lib()
    small, large = (L.lcq_compress_workspace_bytes(q, t, c * 1024) for c in (64, 64 + (1 << 17)))
    assert large - small == (3 * 4 + 2 * 64) * (1 << 17)
