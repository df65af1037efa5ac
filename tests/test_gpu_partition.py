"""The partition of the attention kernel at the edges of its forms.

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
            assert np.array_equal(more[:B].view(np.uint16), got.view(np.uint16)), f"padded to {pad_to}"
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
