"""The append's builds (shifts or divisions, new rows read through the caches or
past them) at the edges of each, bit for bit against the row scatter."""
import numpy as np
import pytest

import apex_workloads as W
from oracle import kv_cache
from test_gpu_kv_append import apex, assert_bitwise, run_append, torch_cuda  # noqa: F401  (fixtures)

pytestmark = pytest.mark.gpu

# (T, NB, Hkv, d, bs): rows around one and two passes of a work group, and each
# of vectors per row, kv-heads and block size not a power of two
SHAPES = [(1, 1, 1, 128, 16), (2, 2, 8, 128, 16), (3, 2, 8, 128, 16), (4, 2, 8, 128, 16), (5, 2, 8, 128, 16),
          (9, 3, 5, 128, 16), (40, 7, 8, 128, 12), (40, 7, 8, 40, 16), (41, 9, 6, 24, 10), (3, 4, 1, 2048, 16),
          (7, 9, 1, 2040, 7)]


@pytest.mark.parametrize("T,NB,Hkv,d,bs", SHAPES)
def test_row_counts_and_shapes(torch_cuda, apex, T, NB, Hkv, d, bs):  # noqa: F811
    c = W.make_append_case(T, NB, Hkv, d, bs, seed=T + d, padding=int(T > 2), out_of_range=int(T > 2))
    gk, gv = run_append(torch_cuda, apex, c)
    rk, rv = kv_cache.kv_append(c.k_cache, c.v_cache, c.k_new, c.v_new, c.slot_mapping)
    assert_bitwise(gk, rk, "k")
    assert_bitwise(gv, rv, "v")


# rows around 128 MiB of new K and V, where they are read past the caches
@pytest.mark.parametrize("T,Hkv,d,bs", [(16384, 1, 2048, 16), (16385, 1, 2048, 16), (5500, 6, 1024, 10)])
def test_large_appends(torch_cuda, apex, T, Hkv, d, bs):  # noqa: F811
    torch = torch_cuda
    g = torch.Generator(device="cuda").manual_seed(T)
    NB = -(-T // bs) + 3
    kv = torch.randint(0, 1 << 15, (T, 2, Hkv, d), generator=g, device="cuda", dtype=torch.int16).view(torch.float16)
    slots = torch.randperm(NB * bs, generator=g, device="cuda")[:T]
    slots[::97] = -1
    caches = [torch.full((NB, Hkv, bs, d), 7, dtype=torch.int16, device="cuda").view(torch.float16) for _ in range(2)]
    apex.kv_append(kv[:, 0], kv[:, 1], caches[0], caches[1], slots)
    used = slots >= 0
    for i in range(2):
        want = torch.full((NB, Hkv, bs, d), 7, dtype=torch.int16, device="cuda")
        want[slots[used] // bs, :, slots[used] % bs] = kv[:, i].view(torch.int16)[used]
        assert torch.equal(caches[i].view(torch.int16), want)


def test_padding_costs_its_slots_only(torch_cuda, apex):  # noqa: F811
    """54 000 tokens of which 95 % are padding: their new rows are not read, so
    the call takes about a ninth of the time without padding (half when every
    row is read).  The best of several runs of ten calls each."""
    torch = torch_cuda
    T, Hkv, d, bs = 54000, 8, 128, 16
    NB = -(-T // bs)
    kv = torch.zeros((T, 2, Hkv, d), dtype=torch.float16, device="cuda")
    caches = [torch.zeros((NB, Hkv, bs, d), dtype=torch.float16, device="cuda") for _ in range(2)]
    full = torch.arange(T, device="cuda")
    padded = torch.where(full < T // 20, full, -1)
    best = {}
    for name, slots in (("full", full), ("padded", padded)) * 5:
        ev = [torch.cuda.Event(enable_timing=True) for _ in range(2)]
        ev[0].record()
        for _ in range(10):
            apex.kv_append(kv[:, 0], kv[:, 1], caches[0], caches[1], slots)
        ev[1].record()
        torch.cuda.synchronize()
        best[name] = min(best.get(name, 1e9), ev[0].elapsed_time(ev[1]) * 100)
    print(f"[append] {T} tokens: {best['full']:.1f} us, 95 % padding {best['padded']:.1f} us", flush=True)
    assert best["padded"] < 0.3 * best["full"]


def test_more_work_groups_than_one_grid_dimension_holds(torch_cuda, apex):  # noqa: F811
    """2^25 + 5 rows of 129 vectors, one row per pass of a work group: more
    threads than a grid dimension counts to.  Nearly all tokens are padding; the
    others are the first, the last and those around the cuts of the grid."""
    torch = torch_cuda
    torch.cuda.empty_cache()
    T, d = (1 << 25) + 5, 1032
    if torch.cuda.mem_get_info()[0] < 80 << 30:
        pytest.skip("needs 70 GB of free device memory")
    new = torch.empty((T, 1, d), dtype=torch.float16, device="cuda")     # K and V: one buffer serves both
    rows = [0, 1, (1 << 23) - 1, 1 << 23, (1 << 24) - 1, 1 << 24, (1 << 24) + 3, (1 << 25) - 1, 1 << 25, T - 1]
    slots = torch.full((T,), -1, dtype=torch.int64, device="cuda")
    want = torch.full((1, 1, 16, d), 9, dtype=torch.float16, device="cuda")
    for i, r in enumerate(rows):
        new[r] = i + 1
        slots[r] = 15 - i
        want[0, 0, 15 - i] = i + 1
    caches = [torch.full((1, 1, 16, d), 9, dtype=torch.float16, device="cuda") for _ in range(2)]
    apex.kv_append(new, new, caches[0], caches[1], slots)
    torch.cuda.synchronize()
    assert torch.equal(caches[0], want) and torch.equal(caches[1], want)
    del new, slots
    torch.cuda.empty_cache()
