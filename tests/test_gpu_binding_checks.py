"""The binding's quick acceptance of its tensors refuses everything the full
checks refuse, argument by argument, with their errors."""
import pytest

import apex_workloads as W
from test_gpu_parity import apex, to_dev, torch_cuda  # noqa: F401  (fixtures)

pytestmark = pytest.mark.gpu

BREAK = {
    "dtype": lambda t: t.to("cuda").double() if t.is_floating_point() else t.long() if str(t.dtype) != "torch.int64" else t.int(),
    "host": lambda t: t.cpu(),
    "shape": lambda t: t[..., :-1].contiguous() if t.dim() > 1 else t[:-1],
    "gaps": lambda t: t.repeat_interleave(2, dim=-1)[..., ::2],
}


def refused(call, args, kw=None):
    with pytest.raises((TypeError, ValueError)):
        call(*args, **(kw or {}))


@pytest.mark.parametrize("how", list(BREAK))
def test_attention_arguments(torch_cuda, apex, how):  # noqa: F811
    torch = torch_cuda
    case = W.make_host_case([40, 17, 100], 8, 2, seed=3)
    good = list(to_dev(torch, case))
    out = torch.empty_like(good[0])
    lse = torch.empty((3, 8), dtype=torch.float32, device="cuda")
    new = torch.zeros((3, 2, 128), dtype=torch.float16, device="cuda")
    base = apex.decode_attention(*good, case.scale)
    for i in range(5):
        if how == "shape" and i == 3:
            continue     # any row width is a table
        bad = list(good)
        bad[i] = BREAK[how](bad[i])
        refused(apex.decode_attention, (*bad, case.scale))
        refused(apex.decode_attention_noalloc, (*bad, case.scale, out))
        refused(apex.decode_attention_ex, (*bad, case.scale))
    refused(apex.decode_attention, (*good, case.scale, BREAK[how](out)))
    refused(apex.decode_attention_noalloc, (*good, case.scale, BREAK[how](out)))
    refused(apex.decode_attention_ex, (*good, case.scale), dict(lse_out=BREAK[how](lse)))
    refused(apex.decode_attention_ex, (*good, case.scale), dict(k_new=BREAK[how](new), v_new=new))
    refused(apex.decode_attention_ex, (*good, case.scale), dict(block_table_stride=good[3].shape[1] + 1))
    assert torch.equal(apex.decode_attention_ex(*good, case.scale, block_table_stride=good[3].shape[1]), base)


@pytest.mark.parametrize("how", list(BREAK))
def test_append_arguments(torch_cuda, apex, how):  # noqa: F811
    torch = torch_cuda
    rows = [torch.zeros((5, 2, 128), dtype=torch.float16, device="cuda") for _ in range(2)]
    caches = [torch.zeros((3, 2, 16, 128), dtype=torch.float16, device="cuda") for _ in range(2)]
    good = [*rows, *caches, torch.arange(5, device="cuda")]
    apex.kv_append(*good)
    for i in range(5):
        bad = list(good)
        bad[i] = BREAK[how](bad[i])
        refused(apex.kv_append, bad)
