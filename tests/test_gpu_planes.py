"""The pruned pass row by row (heavy maps that outgrow the LDS): rows whose cells keep a bit each, rows
folded by two cells to a bit, one cell around each limit, the coarse map beyond (and below four
rows), ragged coordinate counts, both selections, against the full estimate of the same library (itself checked against the oracle
elsewhere) and the oracle's top-k (needs an MI355X)."""
import numpy as np
import pytest

import oracle
import synth
from test_gpu_parity import DEV, host, to_dev

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")
gs = pytest.importorskip("paper_2108_06004_amd")

BITS = (160 * 1024 // 4 - 64) * 32  # cells of a row looked up one bit each


@pytest.mark.parametrize("d,r,c,k", [
    (1_500_037, 5, 300_000, 1_500),       # 1.5M map bits: row by row, no folding
    (900_001, 4, BITS, 900),              # the last width without folding
    (900_001, 4, BITS + 1, 900),          # folded by two, only a little
    (2_000_063, 5, 2 * BITS - 256, 40),   # folded by two throughout
    (2_000_063, 5, 2 * BITS - 255, 2_000),  # the coarse map
    (900_001, 3, BITS + 1, 900),          # three rows: the coarse map
    (700_001, 4, 11_000_003, 700),        # beyond every map in LDS
    (65, 4, 1_400_001, 3),                # fewer coordinates than one wave's pass
    (262_144, 16, 100_000, 262),          # sixteen rows
])
def test_row_by_row_matches(monkeypatch, d, r, c, k):
    monkeypatch.setenv("GS_SELECT_PATH", "pruned")
    hp = synth.hash_params(synth.BASE_SEED + 81 + r, r)
    gen = torch.Generator(device=DEV).manual_seed(d)
    m = torch.randn((r, c), generator=gen, device=DEV)
    m *= torch.exp(2.0 * torch.randn((r, c), generator=gen, device=DEV))  # a heavy tail, so the bound prunes
    ctx = gs.GsContext(d, 1, r, c, k, hp)
    est = torch.empty(d, dtype=torch.float32, device=DEV)
    full, idx = (torch.empty(k, dtype=torch.int32, device=DEV) for _ in range(2))
    ctx.unsketch_topk(m, k, full, est)
    ctx.unsketch_topk(m, k, idx)
    assert np.array_equal(host(full), oracle.topk(host(est), k)[0])
    assert torch.equal(idx, full)
    rng = np.random.default_rng(d)
    rnd = to_dev(rng.integers(0, 1 << 32, d, dtype=np.uint64).astype(np.uint32).view(np.int32))
    nh = [torch.empty(1, dtype=torch.int64, device=DEV) for _ in range(2)]
    ctx.heavymix_topk(m, k, rnd, full, est=est, n_heavy=nh[0])
    ctx.heavymix_topk(m, k, rnd, idx, n_heavy=nh[1])
    assert torch.equal(idx, full) and torch.equal(nh[0], nh[1])
    ctx.close()
