"""The selection's tail (digit passes and emit) on sketches made for its edges: keys many octaves
above the sampled bound, ties from a few to all coordinates (the crowded bin that does not
fit the LDS), one and two digit passes, and one and many emit ranges, all against the oracle's
estimates and top-k bit for bit (the pruned pass falling short of k: test_gpu_input_shapes.py; needs
an MI355X)."""
import numpy as np
import pytest

import oracle
import synth
from test_gpu_parity import DEV, host, to_dev

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")
gs = pytest.importorskip("paper_2108_06004_amd")


def sketch(kind, r, c, rng):
    x = rng.standard_normal((r, c)).astype(np.float32)
    if kind == "octaves":  # a few cells up to 60 octaves above the rest
        hit = rng.random((r, c)) < 0.02
        x[hit] *= np.exp2(rng.uniform(0, 60, int(hit.sum()))).astype(np.float32)
    elif kind == "levels":  # every cell one of eight values: thousands of ties at every key
        x = np.sign(x) * rng.integers(1, 9, (r, c)).astype(np.float32)
    elif kind == "one":  # a single value: every coordinate ties
        x = np.sign(x) * np.float32(0.5)
    elif kind == "tiny":  # subnormal and zero cells
        x = (x * np.float32(1e-40)).astype(np.float32)
        x[rng.random((r, c)) < 0.5] = 0.0
    return np.ascontiguousarray(x.astype(np.float32))


@pytest.mark.parametrize("path", ["pruned", "full"])
@pytest.mark.parametrize("kind", ["normal", "octaves", "levels", "one", "tiny"])
@pytest.mark.parametrize("d,r,c,ks", [
    (4_095, 1, 64, (1, 64, 4_095)),                 # one emit range, one row: d / c ties per cell
    (4_097, 5, 4_097, (1, 257, 4_000)),             # two ranges
    (300_001, 4, 1_000, (3, 3_000, 90_000)),        # ragged ranges, even rows, k past the sampled bound's reach
    (1_100_003, 3, 50_000, (1, 11_000, 600_000)),   # dense: a second digit pass
])
def test_tail_matches_oracle(monkeypatch, path, kind, d, r, c, ks):
    monkeypatch.setenv("GS_SELECT_PATH", path)
    hp = synth.hash_params(synth.BASE_SEED + 61 + d, r)
    rng = np.random.default_rng(d + 7 * r)
    m = sketch(kind, r, c, rng)
    est = oracle.unsketch(m, hp, d)
    ctx = gs.GsContext(d, 1, r, c, max(ks), hp)
    m_d = to_dev(m)
    rnd = rng.integers(0, 1 << 32, d, dtype=np.uint64).astype(np.uint32)
    rnd_d = to_dev(rnd.view(np.int32))
    # the k's in both orders on one context: what a call leaves behind must not matter
    for k in ks + ks[::-1]:
        print(f"[tail] {path} {kind} d={d} r={r} c={c} k={k}", flush=True)
        idx = torch.empty(k, dtype=torch.int32, device=DEV)
        ctx.unsketch_topk(m_d, k, idx)
        assert np.array_equal(host(idx), oracle.topk(est, k)[0]), f"k={k}"
        nh = torch.empty(1, dtype=torch.int64, device=DEV)
        ctx.heavymix_topk(m_d, k, rnd_d, idx, n_heavy=nh)
        ref = oracle.heavymix(m, hp, d, k, rnd)
        assert np.array_equal(host(idx), ref["idx"]) and int(host(nh)[0]) == ref["n_heavy"], f"heavymix k={k}"
    ctx.close()
