"""The full estimate read by tile (k_push and k_median): every row pushed, rows without scratch read
from the table, packed and unpacked lists, tiles split into segments, large selections chosen by
density, against the oracle bit for bit (needs an MI355X)."""
import numpy as np
import pytest

import oracle
import synth
from test_gpu_parity import DEV, host, to_dev

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")
gs = pytest.importorskip("paper_2108_06004_amd")


@pytest.mark.parametrize("sketch_path", ["", "unpacked"])
@pytest.mark.parametrize("layout", ["worker_major", "interleaved"])
@pytest.mark.parametrize("d,P,r,c,k", [
    (1, 2, 1, 1, 1), (4_097, 2, 3, 211, 4_097), (50_001, 1, 5, 5_003, 12_500), (50_001, 3, 8, 5_003, 700),
    (120_011, 6, 9, 900, 30_000), (400_001, 2, 2, 3, 50), (33_333, 20, 16, 4_096, 8_000),
])
def test_tiles_match_oracle(monkeypatch, d, P, r, c, k, layout, sketch_path):
    monkeypatch.setenv("GS_ESTIMATE_PATH", "tiles")
    monkeypatch.setenv("GS_SELECT_PATH", "full")
    if sketch_path:
        monkeypatch.setenv("GS_SKETCH_PATH", sketch_path)
    hp = synth.hash_params(synth.BASE_SEED + 91 + r, r)
    rng = np.random.default_rng(d + r)
    m = rng.standard_normal((r, c)).astype(np.float32)
    ctx = gs.GsContext(d, P, r, c, k, hp, state_layout=layout)
    ref = oracle.unsketch(m, hp, d)
    est = torch.empty(d, dtype=torch.float32, device=DEV)
    idx = torch.empty(k, dtype=torch.int32, device=DEV)
    rnd = rng.integers(0, 1 << 32, d, dtype=np.uint64).astype(np.uint32)
    hm = oracle.heavymix(m, hp, d, k, rnd)
    nh = torch.empty(1, dtype=torch.int64, device=DEV)
    for e in (est, None):  # with and without the estimate vector, twice on one context
        ctx.unsketch_topk(to_dev(m), k, idx, e)
        assert np.array_equal(host(idx), oracle.topk(ref, k)[0])
        assert np.array_equal(host(est), ref)
        ctx.heavymix_topk(to_dev(m), k, to_dev(rnd.view(np.int32)), idx, est=e, n_heavy=nh)
        assert np.array_equal(host(idx), hm["idx"]) and int(host(nh)[0]) == hm["n_heavy"]
    ctx.close()


@pytest.mark.parametrize("c", [60_000, 400_000])  # a table read directly, one read by tile
def test_density_rule(monkeypatch, c):
    # on both sides of the density where a selection estimates every coordinate, on one context
    monkeypatch.delenv("GS_SELECT_PATH", raising=False)
    d, r = 1_000_003, 5
    hp = synth.hash_params(synth.BASE_SEED + 97, r)
    m = np.random.default_rng(98).standard_normal((r, c)).astype(np.float32)
    ref = oracle.unsketch(m, hp, d)
    ctx = gs.GsContext(d, 4, r, c, d, hp)
    for k in (1_000, d // 10, d // 10 + 1, d // 5, d // 5 + 1, d, 7):
        idx = torch.empty(k, dtype=torch.int32, device=DEV)
        ctx.unsketch_topk(to_dev(m), k, idx)
        assert np.array_equal(host(idx), oracle.topk(ref, k)[0]), k
    ctx.close()
