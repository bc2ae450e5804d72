"""The pull with non-temporal list loads (lists beyond 256 MiB, up to four workers): the merged sketch
against 64-bit cell sums of the same state, both state layouts (needs an MI355X)."""
import numpy as np
import pytest

import synth
from test_gpu_parity import DEV

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")
gs = pytest.importorskip("paper_2108_06004_amd")


@pytest.mark.parametrize("P,layout", [(1, "worker_major"), (1, "interleaved"), (2, "interleaved"), (3, "worker_major"),
                                      (4, "interleaved")])
@pytest.mark.parametrize("d", [13_421_800, 13_500_001])  # r d * 4 bytes + padding about and above 2^28
def test_long_lists(d, P, layout):
    r, c = 5, 50_021
    hp = synth.hash_params(synth.BASE_SEED + 71, r)
    gen = torch.Generator(device=DEV).manual_seed(72 + P)
    # integers: every cell sum is exact in fp32 whatever its order, so the tables are compared exactly
    v = torch.randint(-8, 9, (P, d), generator=gen, device=DEV).float()
    ctx = gs.GsContext(d, P, r, c, 10, hp, state_layout=layout)
    tables = torch.empty((P, r, c), dtype=torch.float32, device=DEV)
    ctx.sketch(ctx.to_state(v), tables)
    i = torch.arange(d, dtype=torch.int64, device=DEV)
    p = synth.MERSENNE_P
    for j in range(r):
        col = (i * int(hp["a"][j]) + int(hp["b"][j])) % p % c
        sign = ((i * int(hp["a2"][j]) + int(hp["b2"][j])) % p % 2 * 2 - 1).double()
        for q in range(P):
            ref = torch.zeros(c, dtype=torch.float64, device=DEV).index_add_(0, col, v[q].double() * sign)
            assert torch.equal(tables[q, j].double(), ref), f"worker {q} row {j}"
    ctx.close()
