"""Device memory that an index holds."""
import numpy as np
import pytest

from oracle.oracle import Oracle
from parity import compare_states, say
from workloads import IndexConfig
from workloads.generators import cagra_init_lists

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


def test_a_construction_gives_its_records_back():
    """2,000 points need about 6M records during the construction (some 190
    MiB) and 8,192 for batches of 256; the buffers grow again for a larger
    batch that follows."""
    from paper_2608_21163_amd import GrandIndex

    say("[memory] after a construction")
    n, R, K, S = 2_000, 32, 64, 16
    cfg = IndexConfig("cagra", "f32", "l2", 24, 3_000, R, 64)
    x = np.random.default_rng(7).standard_normal((3_000, 24)).astype(np.float32)
    ids = np.arange(3_000, dtype=np.uint32)
    init = cagra_init_lists(n, K, 8)
    g = GrandIndex.from_config(cfg, max_batch=256)
    _, b = _held(lambda: g.build_cagra(ids[:n], x[:n], init, K, 2, S))
    say(f"  {b / 2**20:.0f} MiB")
    assert b < 48 << 20
    o = Oracle(cfg)
    assert o.build_cagra(ids[:n], x[:n], init, K, 2, S) == 0
    for s in (o, g):
        s.insert(ids[n:], x[n:])
        s.delete(ids[:500])
    assert compare_states(g.export(), o.export(), "cagra") == 0
    g.close()
