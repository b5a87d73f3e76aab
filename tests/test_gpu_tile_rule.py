"""The GEMVs and the few-row tiles form the same sums in the same order, so the rule that picks one of
them does not change a result: the same tokens evaluated in a call on one side of the rule's limit and
in a larger call on the other side give the same bits (ordered combine).  Which kernel each call runs is
asked of the rule itself."""
import pytest
import torch

import oracle
import paper_2608_16157_amd as ftm
import workloads
from tests._util import few_row_tiles, oracle_inputs

pytestmark = pytest.mark.gpu

BF16, FP8, MXFP4 = workloads.DT_BF16, workloads.DT_FP8, workloads.DT_MXFP4
# the bounds of tests/test_gpu_parity.py: one bf16 rounding of h per element, sums in float32
TOL = {BF16: 1e-2, FP8: 3e-2, MXFP4: 1e-2}


def forward(lay, T, act_quant, combine=ftm.FT_COMBINE_ORDERED):
    desc = dict(lay.desc(), act_quant=act_quant, combine=combine)
    ws, route = ftm.alloc_workspace(desc, T), ftm.RouteBuffers(T, lay.top_k, lay.n_experts)
    out = torch.full((T, lay.hidden), float("nan"), device="cuda")
    ftm.ft_moe_forward(desc, ftm.banks_of(lay), lay.logits[:T].contiguous(), lay.slot_table, lay.x[:T].contiguous(), T,
                       out, route, ws)
    torch.cuda.synchronize()
    return out


def kernels(T, H, I, wdt):
    """Few-row tiles (True) or GEMV in the gate/up and in the down projection."""
    return tuple(few_row_tiles([(T, H, I, wdt, 0), (T, H, I, wdt, 1)]))


@pytest.mark.parametrize("wdt,few,many,H,I,changes", [
    # K blocks that split four ways, two ways and neither, in either projection; groups of more than
    # 64 rows in the larger call
    (BF16, 32, 33, 1024, 640, (0, 1)),
    (BF16, 32, 65, 768, 128, (1, 1)),
    (BF16, 64, 200, 640, 1024, (1, 0)),
    (FP8, 16, 17, 1024, 640, (1, 1)),
    (FP8, 5, 160, 768, 128, (1, 1)),
    (FP8, 16, 64, 128, 768, (1, 1)),
    (MXFP4, 3, 4, 1024, 640, (1, 0)),
    (MXFP4, 6, 7, 768, 1024, (0, 1)),
    (MXFP4, 3, 180, 640, 768, (1, 1)),
    # weight rows a multiple of 4096 bytes apart
    (BF16, 95, 96, 2048, 128, (1, 0)),
    (FP8, 95, 96, 4096, 256, (1, 0)),
    (FP8, 95, 96, 128, 4096, (0, 1)),
    (MXFP4, 95, 96, 128, 8192, (0, 1)),
    # the most K the tiles take (64 K blocks), and one block more, which no call below 256 tokens takes
    (FP8, 95, 255, 8192, 128, (1, 0)),
    (FP8, 95, 255, 128, 8192, (0, 1)),
    (BF16, 64, 65, 8064, 128, (1, 0)),
    (BF16, 40, 255, 8320, 128, (0, 0)),
    (MXFP4, 3, 255, 128, 8320, (0, 0)),
])
def test_same_bits_on_both_sides(wdt, few, many, H, I, changes):
    a, b = kernels(few, H, I, wdt), kernels(many, H, I, wdt)
    assert tuple(int(x != y) for x, y in zip(a, b)) == changes
    lay = workloads.random_layer(few + H, hidden=H, inter=I, n_experts=4, top_k=2, tokens=many, w_dtype=wdt, gating=1,
                                 n_resident=4, shared=True, zipf_s=1.0, device="cuda")
    print(f"{wdt} H={H} I={I}: {few} tokens {a}, {many} tokens {b}", flush=True)
    for act in (ftm.FT_ACT_EXACT, ftm.FT_ACT_FP8_1x128_POW2) if wdt == FP8 else (ftm.FT_ACT_EXACT,):
        assert torch.equal(forward(lay, few, act), forward(lay, many, act)[:few])
    ref, _ = oracle.moe_partial(*oracle_inputs(lay), tokens=list(range(0, many, 7)))
    got = forward(lay, many, ftm.FT_ACT_EXACT)[::7].cpu().numpy()
    assert oracle.max_rel_err(got, ref[::7]) <= TOL[wdt]


@pytest.mark.parametrize("wdt,T,H,I,ran", [
    (BF16, 40, 256, 128, (False, True)),
    (MXFP4, 5, 256, 128, (True, False)),
    (FP8, 40, 128, 4096, (True, False)),
])
def test_atomic_combine_of_mixed_kernels(wdt, T, H, I, ran):
    """A GEMV in one projection and tiles in the other: whichever runs first zeroes the output that the other
    adds into."""
    assert kernels(T, H, I, wdt) == ran
    lay = workloads.random_layer(T, hidden=H, inter=I, n_experts=6, top_k=3, tokens=T, w_dtype=wdt, n_resident=5,
                                 shared=True, device="cuda")
    ref, _ = oracle.moe_partial(*oracle_inputs(lay))
    for act in (ftm.FT_ACT_EXACT, ftm.FT_ACT_FP8_1x128_POW2) if wdt == FP8 else (ftm.FT_ACT_EXACT,):
        got = forward(lay, T, act, ftm.FT_COMBINE_ATOMIC)
        torch.testing.assert_close(got, forward(lay, T, act), rtol=1e-5, atol=1e-5 * float(got.abs().max()))
    assert oracle.max_rel_err(forward(lay, T, ftm.FT_ACT_EXACT, ftm.FT_COMBINE_ATOMIC).cpu().numpy(), ref) <= TOL[wdt]
