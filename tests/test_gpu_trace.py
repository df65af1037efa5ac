"""The work-group trace build (libapex_decode_trace.so): the same outputs as
the product library, bit for bit, and a consistent timeline -- every active
work group's prologue, first tiles and end in order, the units of all work
groups adding up to the call's, and each one's segments and units those of the
partition that the host mirrors describe."""
import ctypes

import numpy as np
import pytest

import apex_workloads as W

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch_cuda():
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return torch


def test_trace_build_matches_the_product_and_records_a_timeline(torch_cuda):
    torch = torch_cuda
    import paper_2506_03296_amd as A
    from paper_2506_03296_amd import wg_trace
    product = A.load_library()
    trace = wg_trace.load_trace_library()
    case = W.make_host_case([3000, 17, 900, 4500, 0, 1, 2048], 32, 8, seed=31, poison=True)
    dev = "cuda"
    q, k, v = (torch.from_numpy(x).to(dev) for x in (case.q, case.k_cache, case.v_cache))
    bt, lens = torch.from_numpy(case.block_table).to(dev), torch.from_numpy(case.context_lens).to(dev)
    buf = torch.zeros((4096, wg_trace.WORDS), dtype=torch.int64, device=dev)
    outs = {}
    try:
        for name, lib in (("product", product), ("trace", trace)):
            A._LIB = lib
            if name == "trace":
                assert lib.apex_decode_trace_buffer(ctypes.c_void_p(buf.data_ptr()), 4096) == 0
            for workers in (0, 5):
                outs[(name, workers)] = A.decode_attention_ex(q, k, v, bt, lens, case.scale,
                                                              num_workers=workers)
                torch.cuda.synchronize()
                if name == "trace":
                    rows = buf.cpu().numpy()
                    used = rows[:, 3] > 0
                    units = int(sum(-(-int(L) // 16) for L in case.context_lens if L > 0)) * 8
                    assert int(rows[used, 6].sum()) == units
                    act = used & (rows[:, 6] > 0)
                    r = rows[act]
                    assert np.all(r[:, 0] <= r[:, 1]) and np.all(r[:, 1] <= r[:, 2])
                    assert np.all(r[:, 2] <= r[:, 3]) and np.all(r[:, 4] >= 1)
                    if workers == 5:
                        assert act.sum() == 5
                    buf.zero_()
            if name == "trace":
                assert lib.apex_decode_trace_buffer(None, 0) == 0
    finally:
        A._LIB = product
    for workers in (0, 5):
        a, b = outs[("product", workers)], outs[("trace", workers)]
        assert torch.equal(a.view(torch.int16), b.view(torch.int16)), workers


def traced_rows(torch, lens, Hq, Hkv, append=False):
    """Rows (uint64 words as int64 [W][8]) of one default-grid call of the trace
    build, W the launched work groups."""
    import paper_2506_03296_amd as A
    from paper_2506_03296_amd import wg_trace
    product, lib = A.load_library(), wg_trace.load_trace_library()
    case = W.make_host_case(lens, Hq, Hkv, seed=len(lens), poison=False)
    t = [torch.from_numpy(x).to("cuda") for x in (case.q, case.k_cache, case.v_cache, case.block_table,
                                                  case.context_lens)]
    kw = {}
    if append:
        kw = {n: torch.randn((len(lens), Hkv, 128), device="cuda").half() for n in ("k_new", "v_new")}
    buf = torch.zeros((4096, wg_trace.WORDS), dtype=torch.int64, device="cuda")
    try:
        A._LIB = lib
        assert lib.apex_decode_trace_buffer(ctypes.c_void_p(buf.data_ptr()), 4096) == 0
        A.decode_attention_ex(*t, case.scale, **kw)
        torch.cuda.synchronize()
        assert lib.apex_decode_trace_buffer(None, 0) == 0
    finally:
        A._LIB = product
    rows = buf.cpu().numpy()
    return rows[rows[:, 3] > 0]


def assert_as_planned(rows, lens, Hq, Hkv):
    """The work groups' segments, split segments and units are those of the
    partition that the host mirrors give for the cached lengths `lens`; returns
    which of the three it was."""
    import paper_2506_03296_amd as A
    nb = np.array([-(-L // 16) if L > 0 else 0 for L in lens])
    pairs = np.repeat(nb[nb > 0], Hkv)
    p, n = A.plan_pairs_host(lens, Hq, Hkv, 512, 256), len(rows)
    seg, split, units = rows[:, 4], rows[:, 5], rows[:, 6]
    assert n == 512 and int(units.sum()) == int(pairs.sum())
    if p["active"] == 0:
        line = A.plan_host(lens, Hkv, 512, cus=256)
        assert int(split.sum()) == line["partials"] and not np.any(seg[line["active"]:])
        assert int(seg.sum()) == int(line["contributors"].sum())
        return "line"
    if len(pairs) > 512:
        # run r of 512 pairs goes to the groups' wave r mod 4, a whole one shifted
        # by 77 groups a wave
        group = [(i - (77 * (i // 512 % 4) if (i // 512 + 1) * 512 <= len(pairs) else 0)) % 512
                 for i in range(len(pairs))]
        assert np.array_equal(seg, np.bincount(group, minlength=512)) and not split.any()
        assert np.array_equal(units, np.bincount(group, weights=pairs, minlength=512))
        return "waves"
    # one part of one pair per work group, in order
    want = [min(T, b - k * T) for b, T in zip(nb, p["part_units"]) if b for _ in range(Hkv) for k in range(-(-b // T))]
    cut = [-(-b // T) > 1 for b, T in zip(nb, p["part_units"]) if b for _ in range(Hkv) for k in range(-(-b // T))]
    assert len(want) == p["active"] and np.array_equal(units[:len(want)], want) and not units[len(want):].any()
    assert np.array_equal(seg, units > 0) and np.array_equal(split[:len(want)], cut)
    return "cut"


# (lens, Hq, Hkv, partition): pairs around one per work group (512) and one per
# wave (2048), one to eight requests per lane, requests around the most that the
# partitions by pairs take (256 and 512), block edges, empty requests
PARTITIONS = [
    ("cut_whole_and_split", [1, 255, 256, 257, 300, 0, 513], 8, 2, "cut"),
    ("cut_512_pairs", [100, 7] * 32, 8, 8, "cut"),
    ("cut_256_requests", [20, 3, 33, 16] * 64, 4, 1, "cut"),
    ("line_257_requests", [20, 3, 33, 16] * 64 + [5], 4, 1, "line"),
    ("line_longest_33", [513] + [500] * 31, 32, 16, "line"),
    ("line_large", [2100] * 16, 32, 8, "line"),
    ("waves_513_pairs", [1, 16, 17] * 57, 12, 3, "waves"),
    ("waves_2048_pairs", [33, 5, 60, 128] * 64, 16, 8, "waves"),
    ("waves_2112_pairs_g1", [33, 5, 60, 20] * 16 + [0], 33, 33, "waves"),
    ("waves_period_8", [476] + [18] * 7 + ([300] + [20] * 7) * 10, 32, 32, "waves"),
    ("waves_512_requests", [int(x) for x in np.random.default_rng(4).integers(0, 90, size=512)], 32, 16, "waves"),
    ("line_513_requests", [int(x) for x in np.random.default_rng(4).integers(1, 90, size=513)], 32, 16, "line"),
]


@pytest.mark.parametrize("name,lens,Hq,Hkv,way", PARTITIONS, ids=[c[0] for c in PARTITIONS])
def test_work_groups_take_what_the_host_mirrors_say(torch_cuda, name, lens, Hq, Hkv, way):
    assert assert_as_planned(traced_rows(torch_cuda, lens, Hq, Hkv), lens, Hq, Hkv) == way


# cached lengths (the fused call's are one longer) whose longest request ends on
# a block edge: the current token opens a block that no work group attends
FUSED = [
    ("cut_longest_32", [512] * 3 + [17] * 29, 32, 16, "cut"),
    ("cut_longest_16", [256] * 8 + [40] * 8, 8, 8, "cut"),
    ("waves_longest_32", [512, 16, 16, 16] * 64, 8, 8, "waves"),
    ("waves_longest_16_g2", [256, 31, 0, 15] * 100, 32, 16, "waves"),
    ("waves_longest_1", [16, 3, 9, 1] * 128, 8, 8, "waves"),
    ("line_longest_33", [528] + [500] * 31, 32, 16, "line"),
]


@pytest.mark.parametrize("name,lens,Hq,Hkv,way", FUSED, ids=[c[0] for c in FUSED])
def test_the_fused_append_is_partitioned_by_its_cached_lengths(torch_cuda, name, lens, Hq, Hkv, way):
    rows = traced_rows(torch_cuda, [L + 1 if L else 0 for L in lens], Hq, Hkv, append=True)
    assert assert_as_planned(rows, lens, Hq, Hkv) == way
