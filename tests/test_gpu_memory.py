"""Device memory that an index holds."""
import pytest

from parity import say
from workloads import IndexConfig

pytestmark = pytest.mark.gpu


def _held(make):
    """(index, device bytes that making it took)."""
    import torch

    from paper_2608_21163_amd import GrandIndex

    # what the first index of a process sets up (context, code, scratch) is not counted
    GrandIndex.from_config(IndexConfig("cagra", "u8", "l2", 16, 1_000, 4, 32), max_batch=64).close()
    torch.cuda.synchronize()
    before = torch.cuda.mem_get_info()[0]
    g = make()
    torch.cuda.synchronize()
    return g, before - torch.cuda.mem_get_info()[0]


def test_short_byte_rows_of_a_cagra_pool_are_not_padded():
    from paper_2608_21163_amd import GrandIndex

    say("[memory] 16-byte and 64-byte rows")
    cap = 4_000_000
    held = []
    for dim in (16, 64):
        g, b = _held(lambda: GrandIndex.from_config(IndexConfig("cagra", "u8", "l2", dim, cap, 4, 32), max_batch=64))
        g.close()
        held.append(b)
    say(f"  {held[0] / 2**20:.0f} and {held[1] / 2**20:.0f} MiB")
    assert held[1] - held[0] > 40 * cap
