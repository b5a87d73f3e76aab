"""The GEMV variants of the calls that few-row tiles take in layers with H and I up to 8192, against the CPU
oracle.  One of them is just above 8192 here: 65 K blocks, which split neither two nor four ways, and 66,
which split two ways."""
import pytest

import oracle
import workloads
from tests._util import few_row_tiles, oracle_inputs
from tests.test_gpu_fp8_act import check_output_aq, oracle_aq, run_forward_aq
from tests.test_gpu_parity import check_output, check_route, run_forward

pytestmark = pytest.mark.gpu

BF16, FP8, MXFP4 = workloads.DT_BF16, workloads.DT_FP8, workloads.DT_MXFP4
CASES = [
    # w_dtype, T, k, H, I; the variant in the long projection unless noted
    (BF16, 17, 2, 8320, 128),     # two M tiles a pass, groups of one and of two
    (BF16, 100, 3, 8448, 256),    # groups of more than one pass, K split two ways
    (BF16, 300, 2, 128, 8320),    # the down projection, a call with the matrix-core path's token count
    (BF16, 40, 2, 256, 8448),
    (FP8, 20, 4, 8320, 128),      # gate/up: narrow (80 pairs), two M tiles a pass; down narrow
    (FP8, 20, 4, 8448, 128),      # the same, K split two ways
    (FP8, 24, 8, 8320, 256),      # gate/up: wide (192 pairs), two M tiles a pass
    (FP8, 32, 8, 8448, 256),
    (FP8, 33, 8, 8448, 128),      # gate/up: wide, four M tiles a pass; down: wide, two K blocks a batch
    (FP8, 300, 3, 8320, 128),
    (FP8, 48, 4, 128, 8320),      # down: wide, two K blocks a batch, an odd count
    (FP8, 30, 4, 128, 8448),      # down: narrow
    (FP8, 70, 4, 256, 8448),      # down: wide, K split two ways
    (MXFP4, 17, 4, 8320, 128),    # wide, two M tiles a pass
    (MXFP4, 63, 4, 8448, 128),
    (MXFP4, 64, 4, 8448, 256),    # gate/up: four M tiles a pass
    (MXFP4, 100, 4, 128, 8320),
    (MXFP4, 20, 4, 256, 8448),
    (MXFP4, 5, 2, 8320, 128),     # narrow (10 pairs), one M tile
    (MXFP4, 16, 4, 8448, 256),    # wide, one M tile, two K blocks a batch
]


@pytest.mark.parametrize("wdt,T,k,H,I", CASES)
def test_gemv_variants(wdt, T, k, H, I):
    assert few_row_tiles([(T, H, I, wdt, 0), (T, H, I, wdt, 1)]) == [False, False]
    lay = workloads.random_layer(T + H, hidden=H, inter=I, n_experts=max(6, k), top_k=k, tokens=T, w_dtype=wdt, gating=1,
                                 n_resident=max(6, k) - 1, shared=True, zipf_s=0.7, device="cuda")
    print(f"dtype {wdt} T={T} k={k} H={H} I={I}", flush=True)
    out, route = run_forward(lay)
    ref, r = oracle.moe_partial(*oracle_inputs(lay))
    check_route(route, r, T, k)
    check_output(out, ref, wdt)


@pytest.mark.parametrize("T,H,I", [(20, 8320, 128), (60, 128, 8448)])
def test_gemv_fp8_activations(T, H, I):
    lay = workloads.random_layer(T, hidden=H, inter=I, n_experts=6, top_k=4, tokens=T, w_dtype=FP8, n_resident=6,
                                 shared=True, device="cuda")
    out, _ = run_forward_aq(lay)
    check_output_aq(out, oracle_aq(lay)[0])
