"""The library's cache of device blocks: plans rebuilt in turn allocate once per size, and what
is kept stays bounded.  Seen from outside, through the device's free memory: a block that goes
back to HIP and is allocated again moves it."""
import pytest
import torch

pytestmark = pytest.mark.gpu

KEPT = 16 << 30                                       # bytes of blocks that may stay


@pytest.fixture(scope="module")
def dg(device):
    import paper_2609_01983_amd as dg
    return dg


def _matrix(device, n, deg):
    gen = torch.Generator(device=device).manual_seed(n)
    col = torch.randint(0, n, (n * deg,), device=device, dtype=torch.int32, generator=gen)
    rowptr = (torch.arange(n + 1, device=device) * deg).to(torch.int32)
    return rowptr, col, torch.ones(n * deg, dtype=torch.float32, device=device)


def _plan(dg, A):
    return dg.Plan(*A, seed=0, walks_per_node=4, walk_len=3)


def test_plans_of_several_sizes_in_turn_allocate_once(dg, device):
    # plans of about 15, 61 and 486 MB and scratch blocks of 1, 4 and 235: none serves for another
    sizes = [_matrix(device, 1 << 14, 100), _matrix(device, 1 << 16, 100), _matrix(device, 1 << 19, 100)]
    free = []
    for cycle in range(4):
        for A in sizes:
            _plan(dg, A).destroy()
            torch.cuda.synchronize()
            if cycle >= 2:
                free.append(torch.cuda.mem_get_info()[0])
    assert len(set(free)) == 1, free


def test_kept_blocks_are_bounded(dg, device):
    n, deg, count = 1 << 20, 152, 14                  # 14 plans of 9 bytes an entry: 18.7 GiB
    A = _matrix(device, n, deg)
    plans = [_plan(dg, A) for _ in range(count)]
    torch.cuda.synchronize()
    alive = torch.cuda.mem_get_info()[0]
    for p in plans:
        p.destroy()
    torch.cuda.synchronize()
    assert torch.cuda.mem_get_info()[0] - alive >= count * 9 * n * deg - KEPT
    _plan(dg, A).destroy()                            # and the cache still serves
