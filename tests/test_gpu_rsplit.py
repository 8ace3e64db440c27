"""Resident row-split kernels: FP32 runs of Kv != Ks or square models up to
K = 1024 whose operator rows stay in the registers of a group's workgroups.

They compute the sums of the column-block kernels (a run that takes the
column-block schedule without being pinned to it, from 192 padded rows on)
and of the row-split schedule.  Against the pinned column-block kernels: V and
S bitwise (the same FP32 chains, the same FP64 folds), J and the probe trace
bitwise up to 256 rows of V and to FP64 reassociation (1e-13) above, at the edges of every tile (one to four chains
per wave, 16 to 64 rows, 16 and 32 columns, part-filled last tiles and
groups, Kv != Ks both ways); receivers' Y and statistics and gradients
bitwise.  Two streams of one context give what each gives alone; a captured
run (column blocks) equals an eager one bitwise in V and S.
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


def _run(rom, inst, M, N, n0=0):
    mu = torch.tensor(inst["mu"][:M], dtype=torch.float64, device="cuda")
    V, S = rom.zeros(M)
    V += 1e-3 * torch.tensor(inst["b"], dtype=torch.float32, device="cuda")
    c = torch.tensor(inst["c"], dtype=torch.float32, device="cuda")
    J = torch.zeros(M, dtype=torch.float64, device="cuda")
    y = torch.zeros((N, M), dtype=torch.float64, device="cuda")
    rom.run_rank2(mu, V, S, N, n0=n0, c=c, J=J, y=y)
    rom.check()
    return [t.cpu().numpy() for t in (V, S, J, y)]


@pytest.mark.parametrize("kv,ks,M", [(192, 130, 1), (130, 192, 17), (256, 200, 128), (250, 256, 500), (256, 256, 700),
                                     (300, 280, 33), (64, 512, 16), (512, 500, 129), (512, 40, 250), (512, 512, 500),
                                     (700, 600, 128), (600, 768, 250), (1000, 1024, 100), (1024, 900, 256)])
def test_rsplit_equals_the_column_blocks(columns_table, kv, ks, M):
    inst = synth.round_to(synth.make_instance(kv, ks, M, seed=kv + 3 * ks + M, skew=False), "f32")
    columns_table(kv, ks, M)
    N = 40
    rom, pinned = _rom(inst), _rom(inst, "columns")
    a, b = _run(rom, inst, M, N, n0=5), _run(pinned, inst, M, N, n0=5)
    assert rom.last_schedule == "columns" and pinned.last_schedule == "columns"
    rom.close(); pinned.close()
    assert np.array_equal(a[0], b[0]) and np.array_equal(a[1], b[1])
    tol = 0.0 if kv <= 256 else 1e-13
    assert np.max(np.abs(a[2] - b[2])) <= tol * np.max(np.abs(b[2]))
    assert np.max(np.abs(a[3] - b[3])) <= tol * np.max(np.abs(b[3]))


@pytest.mark.parametrize("kv,ks,M,R,N", [(256, 200, 64, 16, 400), (300, 340, 7, 3, 60)])
def test_rsplit_receivers_equal_the_column_blocks(kv, ks, M, R, N):
    inst = synth.round_to(synth.make_instance(kv, ks, M, seed=kv + M, skew=False), "f32")
    mu = torch.tensor(inst["mu"], dtype=torch.float64, device="cuda")
    C = torch.tensor(np.random.default_rng(1).standard_normal((R, kv)), dtype=torch.float32, device="cuda")
    outs = []
    for sched in ("auto", "columns"):
        rom = _rom(inst, sched)
        V, S = rom.zeros(M)
        o = rom.run_receivers(mu, V, S, N, C)
        rom.check()
        outs.append([t.cpu().numpy() for t in (V, S, o["Y"], o["stats"])])
        rom.close()
    for a, b in zip(*outs):
        assert np.array_equal(a, b)


@pytest.mark.parametrize("kv,ks,M,N", [(200, 256, 40, 90), (256, 500, 130, 50), (450, 300, 130, 50)])
def test_rsplit_adjoint_equals_the_column_blocks(kv, ks, M, N):
    inst = synth.round_to(synth.make_instance(kv, ks, M, seed=kv + M, skew=False), "f32")
    mu = torch.tensor(inst["mu"], dtype=torch.float64, device="cuda")
    c = torch.tensor(inst["c"], dtype=torch.float32, device="cuda")
    outs = []
    for sched in ("auto", "columns"):
        rom = _rom(inst, sched)
        o = rom.adjoint(mu, N, c)
        outs.append({k: v.cpu().numpy() for k, v in o.items()})
        rom.close()
    for k in outs[0]:
        if k == "J" and kv > 256:
            assert np.max(np.abs(outs[0][k] - outs[1][k])) <= 1e-13 * np.max(np.abs(outs[1][k]))
        else:
            assert np.array_equal(outs[0][k], outs[1][k]), k


def test_rsplit_two_streams_of_one_context(columns_table):
    inst = synth.round_to(synth.make_instance(256, 220, 50, seed=6, skew=False), "f32")
    rom = _rom(inst)
    mu = torch.tensor(inst["mu"], dtype=torch.float64, device="cuda")
    V0, S0 = rom.zeros(50)
    rom.run_rank2(mu, V0, S0, 300)
    streams = [torch.cuda.Stream(), torch.cuda.Stream()]
    outs = [rom.zeros(50) for _ in range(4)]
    torch.cuda.synchronize()
    for i, (V, S) in enumerate(outs):
        rom.run_rank2(mu, V, S, 300, stream=streams[i % 2])
    torch.cuda.synchronize()
    rom.check()
    for V, S in outs:
        assert torch.equal(V, V0) and torch.equal(S, S0)
    rom.close()


def test_rsplit_captured_run_equals_the_eager_one(columns_table):
    inst = synth.round_to(synth.make_instance(256, 220, 20, seed=8, skew=False), "f32")
    columns_table(256, 220, 20)
    rom = _rom(inst)
    mu = torch.tensor(inst["mu"], dtype=torch.float64, device="cuda")
    Ve, Se = rom.zeros(20)
    rom.run_rank2(mu, Ve, Se, 80)
    V, S = rom.zeros(20)
    s, g = torch.cuda.Stream(), torch.cuda.CUDAGraph()
    torch.cuda.synchronize()
    with torch.cuda.graph(g, stream=s):
        rom.run_rank2(mu, V, S, 80, stream=s)
    for _ in range(3):
        V.zero_(); S.zero_()
        torch.cuda.synchronize()
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(V, Ve) and torch.equal(S, Se)
        rom.run_rank2(mu, *rom.zeros(20), 7)
        torch.cuda.synchronize()
    rom.close()
