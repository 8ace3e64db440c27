"""Small FP32 models (any pair of Kv, Ks up to 256 but both above 192): the
kernels that give every 32-term chain of the column blocks lanes of its own.

They compute the column blocks' sums, so against the pinned column-block
kernels everything is bitwise the same: V, S, J, the probe trace, receivers
and gradients, at the edges of every size class (one to four blocks of 64
terms, one and four samples per workgroup, a part-filled last workgroup, rows
that end inside a wave, runs that cross a window of source values), also for
a run captured into a graph.
"""
import numpy as np
import pytest

import synth

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu


def _rom(inst, schedule="auto"):
    from paper_2009_11742_amd import Rom
    return Rom(inst["Avs"], inst["Asv"], inst["b"], inst["dt"], state="f32", schedule=schedule)


@pytest.fixture
def columns_table():
    """The autotuner's table with `columns` for every shape the tests run."""
    from paper_2009_11742_amd import tuning
    saved = tuning.entries()

    def put(kv, ks, M):
        up = lambda x: (x + 63) // 64 * 64
        tuning.put(up(kv), up(ks), up(M), "f32", "columns", [1.0, -1, -1, -1, -1])
    yield put
    tuning.clear()
    for e in saved:
        tuning.put(e["kv_pad"], e["ks_pad"], e["m_pad"], e["op"], e["schedule"], e["us"])


def _instance(kv, ks, M):
    return synth.round_to(synth.make_instance(kv, ks, M, seed=kv + 3 * ks + M, skew=False), "f32")


@pytest.mark.parametrize("kv,ks,M", [
    (1, 1, 1), (16, 17, 3), (64, 64, 256), (64, 63, 257), (65, 30, 5), (30, 128, 300), (128, 128, 2),
    (113, 128, 1001), (129, 64, 7), (50, 192, 258), (192, 128, 40), (100, 150, 259), (192, 192, 33), (131, 190, 300),
    (193, 20, 9), (256, 64, 260), (64, 256, 12), (7, 250, 270), (256, 128, 30), (200, 97, 261), (128, 256, 31),
    (70, 193, 300)])
def test_chains_equal_the_column_blocks(columns_table, kv, ks, M):
    inst = _instance(kv, ks, M)
    columns_table(kv, ks, M)
    N = 131
    outs = []
    for schedule in ("auto", "columns"):
        rom = _rom(inst, schedule)
        mu = torch.tensor(inst["mu"], dtype=torch.float64, device="cuda")
        c = torch.tensor(inst["c"], dtype=torch.float32, device="cuda")
        V, S = rom.zeros(M)
        V += 1e-3 * torch.tensor(inst["b"], dtype=torch.float32, device="cuda")
        J = torch.ones(M, dtype=torch.float64, device="cuda")
        y = torch.zeros((N, M), dtype=torch.float64, device="cuda")
        rom.run_rank2(mu, V, S, N, n0=5, c=c, J=J, y=y)
        rom.run_rank2(mu, V, S, 3, n0=5 + N)
        rom.check()
        assert rom.last_schedule == "columns"
        outs.append([t.cpu().numpy() for t in (V, S, J, y)])
        rom.close()
    for a, b in zip(*outs):
        assert np.isfinite(b).all() and np.array_equal(a, b)


@pytest.mark.parametrize("kv,ks,M,R,N", [(100, 64, 20, 4, 100), (130, 192, 300, 3, 70)])
def test_chains_receivers_equal_the_column_blocks(kv, ks, M, R, N):
    inst = _instance(kv, ks, M)
    mu = torch.tensor(inst["mu"], dtype=torch.float64, device="cuda")
    C = torch.tensor(np.random.default_rng(1).standard_normal((R, kv)), dtype=torch.float32, device="cuda")
    outs = []
    for schedule in ("auto", "columns"):
        rom = _rom(inst, schedule)
        V, S = rom.zeros(M)
        o = rom.run_receivers(mu, V, S, N, C)
        outs.append([t.cpu().numpy() for t in (V, S, o["Y"], o["stats"])])
        rom.close()
    for a, b in zip(*outs):
        assert np.array_equal(a, b)


@pytest.mark.parametrize("kv,ks,M,N", [(40, 64, 6, 90), (128, 100, 130, 100), (192, 150, 9, 70), (200, 128, 140, 70)])
def test_chains_adjoint_equals_the_column_blocks(kv, ks, M, N):
    inst = _instance(kv, ks, M)
    mu = torch.tensor(inst["mu"], dtype=torch.float64, device="cuda")
    c = torch.tensor(inst["c"], dtype=torch.float32, device="cuda")
    outs = []
    for schedule in ("auto", "columns"):
        rom = _rom(inst, schedule)
        o = rom.adjoint(mu, N, c)
        outs.append({k: v.cpu().numpy() for k, v in o.items()})
        rom.close()
    for k in outs[0]:
        assert np.array_equal(outs[0][k], outs[1][k]), k


@pytest.mark.parametrize("M", [4, 300])
def test_chains_captured_run_equals_the_eager_one(columns_table, M):
    inst = _instance(90, 70, M)
    columns_table(90, 70, M)
    rom = _rom(inst)
    mu = torch.tensor(inst["mu"], dtype=torch.float64, device="cuda")
    c = torch.tensor(inst["c"], dtype=torch.float32, device="cuda")
    Ve, Se = rom.zeros(M)
    Je = torch.zeros(M, dtype=torch.float64, device="cuda")
    rom.run_rank2(mu, Ve, Se, 80, c=c, J=Je)
    V, S = rom.zeros(M)
    J = torch.zeros(M, dtype=torch.float64, device="cuda")
    s, g = torch.cuda.Stream(), torch.cuda.CUDAGraph()
    torch.cuda.synchronize()
    with torch.cuda.graph(g, stream=s):
        rom.run_rank2(mu, V, S, 80, c=c, J=J, stream=s)
    for _ in range(3):
        V.zero_(); S.zero_(); J.zero_()
        torch.cuda.synchronize()
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(V, Ve) and torch.equal(S, Se) and torch.equal(J, Je)
        rom.run_rank2(mu, *rom.zeros(M), 7)
        torch.cuda.synchronize()
    rom.close()
