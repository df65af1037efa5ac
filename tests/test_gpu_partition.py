"""The partition of the attention kernel at the edges of its forms, the pair
cut of small batches, whole pairs per wave, and the combine of split pairs.

Batches of up to 512 requests are partitioned by every wave in registers (one
request per lane up to 64, four up to 256, eight above), larger ones and
partitions past 32 bits by the work group through LDS.  All give the same ranges, so a batch padded
with empty requests from one form into the next must give the same bits.
"""
import numpy as np
import pytest

import apex_workloads as W
from test_gpu_parity import (FP32_ALLOWANCE, apex, assert_parity, fp16_ulp, run_gpu,  # noqa: F401  (fixtures)
                             torch_cuda)

pytestmark = pytest.mark.gpu


def ragged(B, seed):
    """Contexts of 0 to 5 blocks, block edges among them, one longer request."""
    rng = np.random.default_rng(seed)
    lens = rng.choice([0, 1, 15, 16, 17, 31, 33, 48, 79], size=B)
    lens[rng.integers(0, B)] = 700
    return [int(x) for x in lens]


@pytest.mark.parametrize("Hq,Hkv", [(8, 1), (16, 8), (65, 65)], ids=["one_head", "g2", "65_heads"])
@pytest.mark.parametrize("B", [1, 63, 64, 65, 129, 256, 257, 511])
def test_partition_forms_agree(torch_cuda, apex, oracle_mod, B, Hq, Hkv):  # noqa: F811
    lens = ragged(B, seed=B)
    case = W.make_host_case(lens, Hq, Hkv, seed=B + Hq, poison=True)
    ref = oracle_mod.decode_attention_f64(case.q, case.k_cache, case.v_cache, case.block_table,
                                          case.context_lens, case.scale)
    for workers in (0, 1, 37):
        got = run_gpu(torch_cuda, apex, case, num_workers=workers)
        assert_parity(got, ref, f"B={B} heads {Hq}/{Hkv} workers={workers}")
        assert np.all(got[np.asarray(lens) == 0] == 0)
        for pad_to in (65, 257, 513):
            if pad_to <= B:
                continue
            n = pad_to - B
            table = np.concatenate([case.block_table, np.zeros((n, case.block_table.shape[1]), np.int32)])
            padded = W.HostCase(np.concatenate([case.q, np.ones((n, Hq, 128), np.float16)]), case.k_cache,
                                case.v_cache, table,
                                np.concatenate([case.context_lens, np.zeros(n, np.int32)]), case.scale)
            more = run_gpu(torch_cuda, apex, padded, num_workers=workers)
            # (the default grid partitions some batches by pairs, up to 256
            # and 512 requests: not the same ranges)
            if workers or apex.plan_pairs_host(lens, Hq, Hkv, 512, 256)["active"] == 0:
                assert np.array_equal(more[:B].view(np.uint16), got.view(np.uint16)), f"padded to {pad_to}"
            assert_parity(more[:B], ref, f"padded to {pad_to}")
            assert np.all(more[B:] == 0)


@pytest.mark.parametrize("G", [1, 2, 4, 8])
@pytest.mark.parametrize("workers", [2, 3, 4, 5, 8, 9, 15, 16, 17, 33, 130])
def test_combine_of_a_split_pair(torch_cuda, apex, oracle_mod, G, workers):  # noqa: F811
    """One pair on `workers` work groups (one unit and a bit each): every count
    around what the emitting threads combine on their own (4; G = 1: 4, 8 and 16
    at a time) and around what four waves hold in flight at once (8 or 16),
    several rounds beyond it."""
    torch = torch_cuda
    L = 16 * workers + 5
    case = W.make_host_case([L], G, 1, seed=workers * 8 + G, poison=True)
    assert int(apex.plan_host([L], 1, workers, forced=True)["contributors"].max()) == workers
    ref, lse_ref = oracle_mod.decode_attention_f64(case.q, case.k_cache, case.v_cache, case.block_table,
                                                   case.context_lens, case.scale, return_lse=True)
    lse = torch.zeros((1, G), dtype=torch.float32, device="cuda")
    got = run_gpu(torch_cuda, apex, case, num_workers=workers, lse_out=lse)
    assert_parity(got, ref, f"G={G}, {workers} contributors")
    # fp32 sums of L <= 2085 weights and one logarithm
    assert np.abs(lse.cpu().numpy() - lse_ref).max() <= 1e-5


# (lens, Hq, Hkv, pair cut applies): a pair's blocks around what stays whole
# (16; 32 where parts do not fit), parts around the largest (24), pairs around one per CU (256) and one
# per work group (512), requests in one and in four per lane, long pairs
PAIR_CUTS = [
    ("whole_and_cut", [1, 255, 256, 257, 300, 0, 513], 8, 2, True),
    ("longest_32", [512] * 3 + [17] * 29, 32, 16, True),
    ("longest_33", [513] + [500] * 31, 32, 16, False),
    ("256_pairs", [300] * 32, 32, 8, True),
    ("257_pairs", [300] * 257, 1, 1, False),
    ("258_pairs", [40, 300] * 64 + [16], 8, 2, True),
    ("512_pairs", [100, 7] * 32, 8, 8, True),
    ("520_pairs", [300, 7] * 32 + [9], 8, 8, False),
    ("100_requests", list(range(1, 401, 4)), 16, 2, True),
    ("65_heads", [650, 40], 65, 65, True),
    ("long_pair", [60000], 8, 1, True),
    ("two_long_g1", [40000, 333], 2, 2, True),
    ("parts_of_24", [5760] * 8, 8, 2, True),
    ("one_unit_more", [5760] * 7 + [5761], 8, 2, False),
    ("large", [2100] * 16, 32, 8, False),
]


@pytest.mark.parametrize("name,lens,Hq,Hkv,cut", PAIR_CUTS, ids=[c[0] for c in PAIR_CUTS])
def test_pair_cut(torch_cuda, apex, oracle_mod, name, lens, Hq, Hkv, cut):  # noqa: F811
    torch = torch_cuda
    props = torch.cuda.get_device_properties(0)
    assert (apex.plan_pairs_host(lens, Hq, Hkv, 512, 256)["active"] > 0) == cut
    assert props.multi_processor_count == 256
    case = W.make_host_case(lens, Hq, Hkv, seed=len(lens) + Hq, poison=True)
    ref = oracle_mod.decode_attention_f64(case.q, case.k_cache, case.v_cache, case.block_table,
                                          case.context_lens, case.scale)
    for kw in ({}, dict(check_inputs=True)):
        got = run_gpu(torch_cuda, apex, case, **kw)
        assert_parity(got, ref, f"{name} {kw}")
        assert np.all(got[np.asarray(lens) == 0] == 0)
    assert apex.check_device_error() == 0


def by_waves(apex, lens, Hq, Hkv):  # noqa: F811
    """The default grid gives whole pairs to single waves (lens: the cached
    lengths).  The pair cut needs at most one pair per work group, so more pairs
    than that and a plan by pairs are the waves'."""
    plan = apex.plan_pairs_host(lens, Hq, Hkv, 512, 256)
    pairs = int((np.asarray(lens) > 0).sum()) * Hkv
    return pairs > 512 and plan["active"] == 512 and int(plan["parts"].max()) == 1


# (lens, Hq, Hkv): pairs around one per work group (512) and one per wave
# (2048), each group size, one, four and eight requests per lane, blocks up to
# the largest (32), block edges, empty requests and requests whose only token is
# the current one
SHORT = [
    ("513_pairs", [1, 16, 17] * 57, 12, 3),
    ("536_pairs_g1", [20, 7, 1] * 22 + [9, 0], 8, 8),
    ("2048_pairs", [33, 5, 60, 128] * 64, 16, 8),
    ("2056_pairs", [20, 1, 16, 30] * 64 + [48], 64, 8),
    ("2112_pairs_g1", [33, 5, 60, 20] * 16 + [0], 33, 33),
    ("4100_pairs_g1", [19, 64, 2, 48] * 102 + [7, 31], 10, 10),
    ("ragged_32_blocks", [int(x) for x in np.random.default_rng(3).integers(0, 513, size=300)], 32, 32),
    ("512_requests", [int(x) for x in np.random.default_rng(4).integers(0, 90, size=512)], 32, 16),
]


@pytest.mark.parametrize("name,lens,Hq,Hkv", SHORT, ids=[c[0] for c in SHORT])
def test_short_pairs_per_wave(torch_cuda, apex, oracle_mod, name, lens, Hq, Hkv):  # noqa: F811
    torch = torch_cuda
    assert by_waves(apex, lens, Hq, Hkv)
    case = W.make_host_case(lens, Hq, Hkv, seed=len(lens) + Hq, poison=True)
    ref, lse_ref = oracle_mod.decode_attention_f64(case.q, case.k_cache, case.v_cache, case.block_table,
                                                   case.context_lens, case.scale, return_lse=True)
    empty = np.asarray(lens) == 0
    for kw in ({}, dict(check_inputs=True)):
        lse = torch.zeros((len(lens), Hq), dtype=torch.float32, device="cuda")
        got = run_gpu(torch_cuda, apex, case, lse_out=lse, **kw)
        assert_parity(got, ref, f"{name} {kw}")
        lse = lse.cpu().numpy()
        assert np.all(got[empty] == 0) and np.all(np.isneginf(lse[empty]))
        # fp32 sums of at most 513 weights and one logarithm
        assert np.abs(lse[~empty] - lse_ref[~empty]).max() <= 1e-5
    assert apex.check_device_error() == 0
    # every output is an fp16 neighbour of the exact value, up to fp32 rounding
    assert np.all(np.abs(got[~empty].astype(np.float64) - ref[~empty]) <= fp16_ulp(ref[~empty]) + FP32_ALLOWANCE)


@pytest.mark.parametrize("name,lens,Hq,Hkv", SHORT, ids=[c[0] for c in SHORT])
@pytest.mark.parametrize("check", [False, True])
def test_short_pairs_with_the_fused_append(torch_cuda, apex, oracle_mod, name, lens, Hq, Hkv, check):  # noqa: F811
    """The fused append equals the append followed by the plain call: outputs
    and log-sum-exp to the bar, caches bit for bit (the current slots hold NaN
    before)."""
    torch = torch_cuda
    assert by_waves(apex, lens, Hq, Hkv)
    lens = [L + 1 if L else 0 for L in lens]
    case = W.make_host_case(lens, Hq, Hkv, seed=7 + len(lens), poison=True)
    rng = np.random.default_rng(8)
    kn, vn = (rng.standard_normal((len(lens), Hkv, 128)).astype(np.float16) for _ in range(2))
    k, v = case.k_cache.copy(), case.v_cache.copy()
    k0, v0 = k.copy(), v.copy()
    for b, L in enumerate(lens):
        if L:
            blk, pos = case.block_table[b, (L - 1) // 16], (L - 1) % 16
            k[blk, :, pos], v[blk, :, pos] = kn[b], vn[b]
            k0[blk, :, pos] = v0[blk, :, pos] = np.nan
    ref, lse_ref = oracle_mod.decode_attention_f64(case.q, k, v, case.block_table, case.context_lens, case.scale,
                                                   return_lse=True)
    dev = [torch.from_numpy(x).cuda() for x in (case.q, k0, v0, case.block_table, case.context_lens, kn, vn)]
    lse = torch.zeros((len(lens), Hq), dtype=torch.float32, device="cuda")
    got = apex.decode_attention_ex(*dev[:5], case.scale, k_new=dev[5], v_new=dev[6], check_inputs=check, lse_out=lse)
    got, lse, some = got.cpu().numpy(), lse.cpu().numpy(), np.asarray(lens) > 0
    assert_parity(got, ref, f"{name} fused, check={check}")
    # every output is an fp16 neighbour of the exact value, up to fp32 rounding
    assert np.all(np.abs(got[some].astype(np.float64) - ref[some]) <= fp16_ulp(ref[some]) + FP32_ALLOWANCE)
    # fp32 sums of at most 513 weights and one logarithm
    assert np.abs(lse[some] - lse_ref[some]).max() <= 1e-5 and np.all(np.isneginf(lse[~some]))
    assert np.array_equal(dev[1].cpu().numpy().view(np.uint16), k.view(np.uint16))
    assert np.array_equal(dev[2].cpu().numpy().view(np.uint16), v.view(np.uint16))
    assert not check or apex.check_device_error() == 0


def test_short_pairs_skip_block_ids_outside_the_pool(torch_cuda, apex, oracle_mod):  # noqa: F811
    """A bad id leaves out its block's tokens: the first, a middle, the last
    block of a pair, and a pair that has no other."""
    lens = [40, 16, 64, 33] * 128
    case = W.make_host_case(lens, 2, 2, seed=11, poison=False)
    assert by_waves(apex, lens, 2, 2)
    bad = {0: 0, 1: 0, 2: 2, 3: 2, 511: 1, 262: 0}
    keep = case.block_table.copy()
    for b, i in bad.items():
        case.block_table[b, i] = -5 if b % 2 else case.k_cache.shape[0]
    got = run_gpu(torch_cuda, apex, case, check_inputs=True)
    assert apex.check_device_error() == apex.DEVICE_ERR_BLOCK_ID
    case.block_table[:] = keep
    for b, L in enumerate(lens):
        tok = np.arange(L)
        if b in bad:
            tok = tok[tok // 16 != bad[b]]
        ids = keep[b, tok // 16]
        kk, vv = (c[ids, :, tok % 16].astype(np.float64) for c in (case.k_cache, case.v_cache))
        for h in range(2):
            s = kk[:, h] @ case.q[b, h].astype(np.float64) * float(case.scale)
            w = np.exp(s - s.max()) if len(s) else s
            want = (w[:, None] * vv[:, h]).sum(0) / w.sum() if len(s) else np.zeros(128)
            assert np.abs(got[b, h] - want).max() <= 2e-3, (b, h)


@pytest.mark.parametrize("Hq,Hkv", [(4, 4), (16, 2)])
def test_short_pairs_keep_infinite_values(torch_cuda, apex, oracle_mod, Hq, Hkv):  # noqa: F811
    """An infinite value in the current token's V row (its weight is positive)
    gives that infinity in its dim, as the cost line does; the other dims are
    what they are without it."""
    torch = torch_cuda
    lens = [17, 33, 20, 50] * (1024 // (4 * Hkv))
    assert by_waves(apex, [L - 1 for L in lens], Hq, Hkv)
    case = W.make_host_case(lens, Hq, Hkv, seed=5, poison=False)
    rng = np.random.default_rng(9)
    kn, vn = (rng.standard_normal((len(lens), Hkv, 128)).astype(np.float16) for _ in range(2))
    vn[0, 0, 0], vn[7, -1, 127], vn[-1, 0, 64] = np.inf, -np.inf, np.inf
    want = np.repeat(np.where(np.isinf(vn), vn, np.float16(0)), Hq // Hkv, axis=1)
    k, v = case.k_cache.copy(), case.v_cache.copy()
    for b, L in enumerate(lens):
        blk, pos = case.block_table[b, (L - 1) // 16], (L - 1) % 16
        k[blk, :, pos], v[blk, :, pos] = kn[b], np.where(np.isinf(vn[b]), np.float16(0), vn[b])
    ref = oracle_mod.decode_attention_f64(case.q, k, v, case.block_table, case.context_lens, case.scale)
    for kw in ({}, dict(num_workers=512)):   # pairs by waves; an explicit grid is cut on the line
        dev = [torch.from_numpy(x).cuda() for x in (case.q, case.k_cache, case.v_cache, case.block_table,
                                                    case.context_lens, kn, vn)]
        got = apex.decode_attention_ex(*dev[:5], case.scale, k_new=dev[5], v_new=dev[6], **kw).cpu().numpy()
        assert not np.isnan(got).any(), kw
        assert np.array_equal(np.where(np.isinf(got), got, np.float16(0)), want), kw
        assert_parity(np.where(want == 0, got, ref.astype(np.float16)), ref, f"finite values, {kw}")
