"""Worker counts whose rows have a partial last 16-byte group or more than sixteen workers, at the
edges of their kernels: the chunks of the interleaved accumulation (64 / G coordinates, four or
eight per pass), the 64- and 256-coordinate chunks of the wide worker-major one, the pull's lane
groups, its segments and its unpacked lists, against the oracle (needs an MI355X)."""
import numpy as np
import pytest

import oracle
import synth
from test_gpu_parity import DEV, Dev, assert_tol, chain_check, host, to_dev

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")
gs = pytest.importorskip("paper_2108_06004_amd")


@pytest.mark.parametrize("layout", ["interleaved", "worker_major"])
@pytest.mark.parametrize("d,P,r,c,k", [
    (1, 17, 3, 1, 1), (63, 6, 3, 9, 5), (129, 2, 3, 40, 9), (255, 13, 4, 31, 255), (256, 20, 5, 33, 7),
    (257, 31, 5, 64, 40), (4_097, 64, 3, 300, 100), (7_919, 33, 5, 211, 90), (20_011, 5, 5, 3_001, 200),
    (33_000, 48, 2, 1_000, 333), (70_001, 61, 3, 2_048, 700), (400_001, 18, 2, 3, 50),
])
def test_worker_count_edges(layout, d, P, r, c, k):
    hp = synth.hash_params(synth.BASE_SEED + 41 * d + P, r)
    rng = np.random.default_rng(d * 43 + P)
    dv = Dev(d, P, r, c, k, hp, 0.9, layout=layout)
    if c == 3:
        assert dv.ctx.describe()["segments"] > 1  # the partials of a split tile are merged per worker
    u = rng.standard_normal((P, d)).astype(np.float32)
    v = rng.standard_normal((P, d)).astype(np.float32)
    for t in range(2):
        g = rng.laplace(0, 1e-2, (P, d)).astype(np.float32)
        u, v = chain_check(dv, g, u, v, k, 0.9, label=f"{layout} d={d} P={P} r={r} c={c} k={k} t={t}")
    dv.close()


def test_wide_unpacked_lists(monkeypatch):
    monkeypatch.setenv("GS_SKETCH_PATH", "unpacked")
    d, P, r, c, k = 9_001, 27, 3, 777, 80
    hp = synth.hash_params(synth.BASE_SEED + 47, r)
    rng = np.random.default_rng(48)
    dv = Dev(d, P, r, c, k, hp, 0.9, layout="interleaved")
    assert dv.ctx.describe()["packed_lists"] == 0
    u, v = (rng.standard_normal((P, d)).astype(np.float32) for _ in range(2))
    g = rng.laplace(0, 1e-2, (P, d)).astype(np.float32)
    chain_check(dv, g, u, v, k, 0.9, label="wide unpacked")
    dv.close()


@pytest.mark.parametrize("P", [1, 6, 22])
def test_padding_keeps_its_bits_and_wide_rows_need_no_alignment(P):
    # every padding entry holds a NaN with a payload, which must survive bit for bit; with more
    # than sixteen workers the state may start at any float (no row copy)
    d, r, c, k = 5_003, 3, 400, 150
    hp = synth.hash_params(synth.BASE_SEED + 53 + P, r)
    rng = np.random.default_rng(54 + P)
    g, u0, v0 = (rng.standard_normal((P, d)).astype(np.float32) for _ in range(3))
    ref = oracle.step(g, u0.copy(), v0.copy(), hp, c, k, rho=0.9, want_tables=False)
    PP = gs.state_stride(P)
    mark = 0x7FC12345
    dv = Dev(d, P, r, c, k, hp, 0.9, layout="interleaved")
    for offset in (0, 1, 3) if P > 16 else (0,):
        bufs = [torch.full((d * PP + offset,), mark, dtype=torch.int32, device=DEV) for _ in range(2)]
        u_d, v_d = (b[offset:].view(torch.float32).view(d, PP) for b in bufs)
        u_d[:, :P] = to_dev(u0).t()
        v_d[:, :P] = to_dev(v0).t()
        dv.ctx.step(to_dev(g), u_d, v_d, k, dv.merged, dv.idx, dv.values)
        uh, vh = host(u_d), host(v_d)
        for x in (uh, vh):
            assert np.all(x[:, P:].copy().view(np.int32) == mark), "padding changed"
        uc, vc = u0.copy(), v0.copy()
        oracle.accumulate(g, uc, vc, 0.9)
        assert np.array_equal(host(dv.values), oracle.gather_reset(host(dv.idx), uc, vc, True))
        assert np.array_equal(uh[:, :P].T, uc) and np.array_equal(vh[:, :P].T, vc)
        assert_tol(host(dv.merged), ref["merged"], f"P={P} offset={offset}")
    dv.close()
