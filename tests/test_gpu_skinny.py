"""The grouped GEMM's tiles of few rows against the CPU oracle, at the edges where they change:
groups of 1 to 65 rows (16-row and 32-row MFMA tiles, the largest skinny group, the first large one),
K extents shorter than, equal to and longer than the staging ring, both combine modes, and calls just
above the streaming kernels' token range."""
import numpy as np
import pytest
import torch

import oracle
import paper_2608_16157_amd as ftm
import workloads
from tests._util import oracle_inputs

pytestmark = pytest.mark.gpu

# the bounds of tests/test_gpu_parity.py: one bf16 rounding of h per element, sums in float32
TOL = {workloads.DT_BF16: 1e-2, workloads.DT_FP8: 3e-2, workloads.DT_MXFP4: 1e-2}


def layer_with_groups(sizes, wdt, hidden, inter, shared, seed=3):
    """One routed expert per token, expert e with sizes[e] tokens scattered over the batch."""
    E, T = len(sizes) + 1, sum(sizes)
    lay = workloads.random_layer(seed, hidden=hidden, inter=inter, n_experts=E, top_k=1, tokens=T,
                                 w_dtype=wdt, gating=1, n_resident=E, shared=shared)
    owner = np.repeat(np.arange(len(sizes)), sizes)
    rng = np.random.default_rng(seed)
    rng.shuffle(owner)
    logits = rng.normal(size=(T, E)).astype(np.float32)
    logits[np.arange(T), owner] += 20.0
    lay.logits = torch.from_numpy(logits)
    return lay.to("cuda")


def check(lay, sizes, combine):
    T = lay.tokens
    desc = dict(lay.desc(), combine=combine)
    ws, route = ftm.alloc_workspace(desc, T), ftm.RouteBuffers(T, lay.top_k, lay.n_experts)
    out = torch.full((T, lay.hidden), float("nan"), device="cuda")
    ftm.ft_moe_forward(desc, ftm.banks_of(lay), lay.logits, lay.slot_table, lay.x, T, out, route, ws)
    torch.cuda.synchronize()
    ref, r = oracle.moe_partial(*oracle_inputs(lay))
    got_sizes = np.diff(r["hit_off"])
    assert sorted(got_sizes[got_sizes > 0].tolist()) == sorted(sizes)
    assert np.array_equal(route.hit_pairs.cpu().numpy()[: r["n_hit"]], r["hit_pairs"])
    assert np.array_equal(route.hit_off.cpu().numpy(), r["hit_off"])
    err = oracle.max_rel_err(out.cpu().numpy(), ref)
    print(f"T={T} {err:.3e}", flush=True)
    assert err <= TOL[lay.w_dtype]


@pytest.mark.parametrize("wdt", [workloads.DT_BF16, workloads.DT_FP8, workloads.DT_MXFP4])
@pytest.mark.parametrize("sizes,hidden,inter,shared,combine", [
    # every tile kind in one call; the shared expert's 228 rows are a large group
    ([1, 16, 17, 32, 33, 64, 65], 256, 128, True, ftm.FT_COMBINE_ORDERED),
    ([1, 16, 17, 32, 33, 64, 65], 768, 640, False, ftm.FT_COMBINE_ATOMIC),
    # skinny groups only, the shared expert's among them
    ([2, 31], 512, 384, True, ftm.FT_COMBINE_ORDERED),
    # one row a group; K blocks that split neither two nor four ways (one and five)
    ([1, 1, 2], 128, 640, True, ftm.FT_COMBINE_ORDERED),
    # large groups only; the most tokens below the matrix-core path's workspace
    ([127, 128], 256, 256, False, ftm.FT_COMBINE_ORDERED),
    # many-token call: skinny and large groups from the many-workgroup router
    ([5, 16, 40, 64, 66, 129, 700], 512, 256, True, ftm.FT_COMBINE_ORDERED),
])
def test_group_sizes(wdt, sizes, hidden, inter, shared, combine):
    check(layer_with_groups(sizes, wdt, hidden, inter, shared), sizes, combine)


def test_fp8_zero_scale_blocks():
    """Blocks of scale 0 contribute nothing, whatever their codes hold (NaN codes among them)."""
    sizes = [3, 20, 50]
    lay = layer_with_groups(sizes, workloads.DT_FP8, 512, 256, False)
    slot = int(lay.slot_table[0])
    for s in range(lay.n_slots):
        lay.s13[s, 0, 1] = 0
        lay.s2[s, 1, 0] = 0
    ref, _ = oracle.moe_partial(*oracle_inputs(lay))
    lay.w13[slot, :128, 128:256] = 0x7F
    T = lay.tokens
    ws, route = ftm.alloc_workspace(lay.desc(), T), ftm.RouteBuffers(T, 1, lay.n_experts)
    out = torch.empty(T, lay.hidden, device="cuda")
    ftm.ft_moe_forward(lay.desc(), ftm.banks_of(lay), lay.logits, lay.slot_table, lay.x, T, out, route, ws)
    torch.cuda.synchronize()
    assert oracle.max_rel_err(out.cpu().numpy(), ref) <= TOL[workloads.DT_FP8]
