"""The largest call: 1048576 tokens, 64 experts a token and the shared one.  Its down projection has more
tiles than one grid dimension holds threads for (2^32)."""
import pytest
import torch

import oracle
import paper_2608_16157_amd as ftm
import workloads
from tests._util import oracle_inputs, to_np_bits

pytestmark = pytest.mark.gpu

BYTES = 90e9   # x 17 GB, the output 34 GB, h 18 GB, lists and rows 5 GB, the generator's float32 block


def test_largest_call():
    if torch.cuda.mem_get_info()[0] < BYTES:
        pytest.skip("needs 90 GB of device memory")
    T, k, H, I = 1048576, 64, 8192, 128
    lay = workloads.random_layer(3, hidden=H, inter=I, n_experts=k, top_k=k, tokens=1, w_dtype=workloads.DT_BF16,
                                 n_resident=k, shared=True, device="cuda")
    g = torch.Generator(device="cuda")
    g.manual_seed(4)
    logits = torch.randn(T, k, generator=g, device="cuda")
    x = torch.empty(T, H, dtype=torch.bfloat16, device="cuda")
    for t in range(0, T, 65536):
        x[t:t + 65536] = torch.randn(65536, H, generator=g, device="cuda")
    desc = lay.desc()
    ws, route = ftm.alloc_workspace(desc, T), ftm.RouteBuffers(T, k, k)
    out = torch.full((T, H), float("nan"), device="cuda")
    ftm.ft_moe_forward(desc, ftm.banks_of(lay), logits, lay.slot_table, x, T, out, route, ws)
    torch.cuda.synchronize()
    # rows of the first, a middle and the last token tiles, against the oracle's layer of those tokens
    rows = torch.tensor([0, 127, 128, 400001, T - 129, T - 1], device="cuda")
    d, banks, _, slots, _ = oracle_inputs(lay)
    ref, _ = oracle.moe_partial(d, banks, to_np_bits(logits[rows]), slots, to_np_bits(x[rows]))
    err = oracle.max_rel_err(out[rows].cpu().numpy(), ref)
    print(f"{err:.3e}", flush=True)
    assert err <= 1e-2
    for t in range(0, T, 65536):   # every tile was written
        assert bool(out[t:t + 65536].isfinite().all())
    del ws, route, out, x, logits
    torch.cuda.empty_cache()
