"""A 128 x 128 block of fp8 weights whose scale is 0 contributes nothing, whatever its codes hold (NaN
codes here), in every kernel that evaluates fp8 layers: the GEMVs of few tokens and of H or I above
8192, the few-row tiles and the matrix-core tiles, with exact and with fp8 activations."""
import pytest
import torch

import oracle
import workloads
from tests._util import oracle_inputs
from tests.test_gpu_fp8_act import check_output_aq, oracle_aq, run_forward_aq
from tests.test_gpu_parity import check_output, run_forward

pytestmark = pytest.mark.gpu


def zero_blocks(w, s, seed):
    """Scale 0 for a third of the blocks of each matrix, the first and the last of a row of blocks among
    them; returns the mask of their codes."""
    g = torch.Generator().manual_seed(seed)
    z = torch.rand(s.shape, generator=g) < 1 / 3
    z[:, 0, 0] = z[:, -1, -1] = True
    s[z.to(s.device)] = 0
    return z.repeat_interleave(128, 1).repeat_interleave(128, 2).to(w.device)


@pytest.mark.parametrize("fp8_act", [False, True])
@pytest.mark.parametrize("T,E,k,H,I", [
    (1, 70, 4, 384, 256),     # routed inside the GEMV; an odd count of K blocks, two a batch
    (5, 8, 3, 512, 384),      # narrow items
    (16, 32, 12, 640, 256),   # wide items, one M tile
    (20, 8, 3, 512, 384),     # few-row tiles
    (20, 8, 3, 8320, 128),    # GEMVs beyond the tiles' tables: narrow, two M tiles a pass
    (60, 6, 3, 128, 8320),    # wide down items, four M tiles a pass in gate/up
    (300, 8, 3, 512, 384),    # matrix-core tiles
])
def test_zero_scale_nan_codes(T, E, k, H, I, fp8_act):
    lay = workloads.random_layer(T + H, hidden=H, inter=I, n_experts=E, top_k=k, tokens=T,
                                 w_dtype=workloads.DT_FP8, gating=1, n_resident=E, shared=True, device="cuda")
    m13, m2 = zero_blocks(lay.w13, lay.s13, 1), zero_blocks(lay.w2, lay.s2, 2)
    lay.w13[m13], lay.w2[m2] = 0, 0
    ref, _ = oracle_aq(lay) if fp8_act else oracle.moe_partial(*oracle_inputs(lay))
    lay.w13[m13], lay.w2[m2] = 0x7F, 0xFF
    out, _ = (run_forward_aq if fp8_act else run_forward)(lay)
    print(f"T={T} H={H} I={I} fp8_act={fp8_act}", flush=True)
    if fp8_act:
        check_output_aq(out, ref)
    else:
        check_output(out, ref, lay.w_dtype)
