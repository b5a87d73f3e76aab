"""Routing of prompt chunks whose blocks each scan the block table for themselves, bit-exact against
the oracle at the edges of its range: the fewest pairs beyond the one-workgroup router, a ragged last
block, the most blocks and one more, one to many experts per scanning thread, 64 pairs per token."""
import pytest
import torch

import oracle
import workloads
from tests._util import oracle_inputs
from tests.test_gpu_parity import check_route, run_route

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("E,k,T,shared,ties", [
    (64, 64, 33, True, False),      # 64 pairs per token
    (128, 8, 257, False, True),
    (3, 3, 700, True, False),       # many scanning threads per expert
    (1000, 5, 500, True, False),    # one scanning thread per expert
    (256, 6, 2048, False, False),   # 32 rows of the table per scanning thread
    (256, 6, 2049, True, False),    # a second batch of rows
    (256, 6, 4096, False, False),   # 256 blocks
    (1024, 2, 4096, True, False),   # all 256 rows by one thread per expert
    (8, 2, 4095, False, True),      # 128 scanning threads per expert
    (128, 8, 4097, True, False),    # one block too many
])
def test_route_place(E, k, T, shared, ties):
    lay = workloads.random_layer(E + T, hidden=128, inter=128, n_experts=E, top_k=k, tokens=T,
                                 w_dtype=workloads.DT_BF16, n_resident=min(E, 40), shared=shared, zipf_s=1.0,
                                 tie_logits=ties, device="cuda")
    inp = oracle_inputs(lay)
    check_route(run_route(lay), oracle.route(inp[0], inp[2], inp[3]), T, k)


def test_route_place_faulty_slot_table():
    T, k, E = 300, 8, 32
    lay = workloads.random_layer(9, hidden=128, inter=128, n_experts=E, top_k=k, tokens=T,
                                 w_dtype=workloads.DT_BF16, n_resident=20, shared=True, device="cuda")
    lay.slot_table[:4] = torch.tensor([5, 5, -7, lay.n_slots - 1], dtype=torch.int32)   # twice, range, shared
    inp = oracle_inputs(lay)
    r = oracle.route(inp[0], inp[2], inp[3])
    assert r["status"] != 0
    check_route(run_route(lay), r, T, k)
