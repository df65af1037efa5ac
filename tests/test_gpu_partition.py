"""The partition of the attention kernel at the edges of its forms, the pair
cut of small batches, and the combine of split pairs.

Batches of up to 256 requests are partitioned by every wave in registers (one
request per lane up to 64, four above), larger ones and partitions past 32 bits
by the work group through LDS.  All give the same ranges, so a batch padded
with empty requests from one form into the next must give the same bits.
"""
import numpy as np
import pytest

import apex_workloads as W
from test_gpu_parity import apex, assert_parity, run_gpu, torch_cuda  # noqa: F401  (fixtures)

pytestmark = pytest.mark.gpu


def ragged(B, seed):
    """Contexts of 0 to 5 blocks, block edges among them, one longer request."""
    rng = np.random.default_rng(seed)
    lens = rng.choice([0, 1, 15, 16, 17, 31, 33, 48, 79], size=B)
    lens[rng.integers(0, B)] = 700
    return [int(x) for x in lens]


@pytest.mark.parametrize("Hq,Hkv", [(8, 1), (16, 8), (65, 65)], ids=["one_head", "g2", "65_heads"])
@pytest.mark.parametrize("B", [1, 63, 64, 65, 129, 256, 257])
def test_partition_forms_agree(torch_cuda, apex, oracle_mod, B, Hq, Hkv):  # noqa: F811
    lens = ragged(B, seed=B)
    case = W.make_host_case(lens, Hq, Hkv, seed=B + Hq, poison=True)
    ref = oracle_mod.decode_attention_f64(case.q, case.k_cache, case.v_cache, case.block_table,
                                          case.context_lens, case.scale)
    for workers in (0, 1, 37):
        got = run_gpu(torch_cuda, apex, case, num_workers=workers)
        assert_parity(got, ref, f"B={B} heads {Hq}/{Hkv} workers={workers}")
        assert np.all(got[np.asarray(lens) == 0] == 0)
        for pad_to in (65, 257):
            if pad_to <= B:
                continue
            n = pad_to - B
            table = np.concatenate([case.block_table, np.zeros((n, case.block_table.shape[1]), np.int32)])
            padded = W.HostCase(np.concatenate([case.q, np.ones((n, Hq, 128), np.float16)]), case.k_cache,
                                case.v_cache, table,
                                np.concatenate([case.context_lens, np.zeros(n, np.int32)]), case.scale)
            more = run_gpu(torch_cuda, apex, padded, num_workers=workers)
            # (the default grid cuts a small batch of up to 256 requests by
            # pairs and never a larger one: not the same ranges)
            if workers or apex.plan_pairs_host(lens, Hq, Hkv, 512, 256)["active"] == 0:
                assert np.array_equal(more[:B].view(np.uint16), got.view(np.uint16)), f"padded to {pad_to}"
            assert_parity(more[:B], ref, f"padded to {pad_to}")
            assert np.all(more[B:] == 0)


@pytest.mark.parametrize("G", [1, 2, 4, 8])
@pytest.mark.parametrize("workers", [2, 3, 4, 5, 15, 16, 17, 33, 130])
def test_combine_of_a_split_pair(torch_cuda, apex, oracle_mod, G, workers):  # noqa: F811
    """One pair on `workers` work groups (one unit and a bit each): every count
    around what the emitting threads combine on their own (4) and around what
    four waves hold in flight at once (8 or 16), several rounds beyond it."""
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
# (16) and around the largest part (32), pairs around one per CU (256) and one
# per work group (512), requests in one and in four per lane, long pairs
PAIR_CUTS = [
    ("whole_and_cut", [1, 255, 256, 257, 300, 0, 513], 8, 2, True),
    ("longest_32", [512] * 3 + [17] * 29, 32, 16, True),
    ("longest_33", [513] + [500] * 31, 32, 16, False),
    ("256_pairs", [300] * 32, 32, 8, True),
    ("257_pairs", [300] * 257, 1, 1, False),
    ("258_pairs", [40, 300] * 64 + [16], 8, 2, True),
    ("512_pairs", [100, 7] * 32, 8, 8, True),
    ("520_pairs", [100, 7] * 32 + [9], 8, 8, False),
    ("100_requests", list(range(1, 401, 4)), 16, 2, True),
    ("65_heads", [700, 40], 65, 65, True),
    ("long_pair", [60000], 8, 1, True),
    ("two_long_g1", [40000, 333], 2, 2, True),
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
