"""States that are not finite through the row-split kernels' exchange, whose
empty slots are a bit pattern (all ones in a 32-bit word, in the high word of
an FP64 one): a state may hold that pattern too, and a run may overflow.

Samples with such states end as NaN or infinity like on the column blocks, the
others keep their bits, and no wait runs out: a row-split run reports none, and
the runs that repeat themselves take far less than a wait that runs out
(2^20 polls, about half a second).
"""
import time

import numpy as np
import pytest

import synth
from paper_2009_11742_amd import _lib

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu


@pytest.fixture
def columns_table():
    """The autotuner's table with `columns` for a shape."""
    from paper_2009_11742_amd import tuning
    tuning.load_default()
    saved = tuning.entries()

    def put(kv, ks, M):
        up = lambda x: (x + 63) // 64 * 64
        tuning.put(up(kv), up(ks), up(M), "f32", "columns", [1.0, -1, -1, -1, -1])
    yield put
    tuning.clear()
    for e in saved:
        tuning.put(e["kv_pad"], e["ks_pad"], e["m_pad"], e["op"], e["schedule"], e["us"])


def _rom(inst, state, schedule, ops=None, dt=None):
    from paper_2009_11742_amd import Rom
    kw = {"ops": ops} if ops else {}
    return Rom(inst["Avs"], inst["Asv"], inst["b"], dt or inst["dt"], state=state, schedule=schedule, **kw)


def _states(rom, inst, M, bad):
    """A state per sample; `bad` samples hold the empty pattern in two
    neighbouring entries of V or of S."""
    g = np.random.default_rng(5)
    t = rom.torch_dtype
    V = torch.tensor(g.standard_normal((M, rom.kv)) * 1e-2, dtype=t, device="cuda")
    S = torch.tensor(g.standard_normal((M, rom.ks)) * 1e-2, dtype=t, device="cuda")
    it = torch.int64 if t == torch.float64 else torch.int32
    for i, m in enumerate(bad):
        X = (V, S)[i % 2]
        X.view(it)[m, 4 * i:4 * i + 2] = -1
    return V, S


def _run(rom, inst, V, S, N):
    M = V.shape[0]
    mu = torch.tensor(inst["mu"], dtype=torch.float64, device="cuda")
    c = torch.tensor(inst["c"], dtype=rom.torch_dtype, device="cuda")
    J = torch.zeros(M, dtype=torch.float64, device="cuda")
    y = torch.zeros((N, M), dtype=torch.float64, device="cuda")
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    rom.run_rank2(mu, V, S, N, c=c, J=J, y=y)
    torch.cuda.synchronize()
    dt = time.perf_counter() - t0
    rom.check()
    return [x.cpu().numpy() for x in (V, S, J, y)], dt


def _compare(x, z, tol):
    """The same entries not finite, BAD samples all of them and no others, the
    rest within tol (0: bitwise) of the largest."""
    f = np.isfinite(z)
    assert np.array_equal(f, np.isfinite(x))
    if tol == 0.0:
        assert np.array_equal(x[f], z[f])
    else:
        assert np.max(np.abs(x[f] - z[f])) <= tol * np.max(np.abs(z[f]))
    whole = f.reshape(len(f), -1).all(axis=1)
    assert sorted(np.flatnonzero(~whole)) == BAD


BAD = [0, 3, 17, 20]


# FP64 row-split kernels against the vector-ALU blocks; FP32 column-block runs
# on the resident row-split kernels against the column-block kernels.
@pytest.mark.parametrize("state,kv,ks,M", [("f64", 128, 128, 21), ("f64", 300, 280, 22), ("f64", 192, 192, 500),
                                           ("f32", 256, 256, 21), ("f32", 300, 280, 40), ("f32", 500, 1000, 33)])
def test_empty_pattern_in_states(columns_table, state, kv, ks, M):
    inst = synth.round_to(synth.make_instance(kv, ks, M, seed=kv + M, skew=False), "f32")
    columns_table(kv, ks, M)
    N = 40
    outs = []
    for schedule in ("auto", "columns"):
        rom = _rom(inst, state, schedule)
        _run(rom, inst, *_states(rom, inst, M, []), N)          # packs, workspace
        out, dt = _run(rom, inst, *_states(rom, inst, M, BAD), N)
        if schedule == "auto":
            assert _lib.load().rom_debug_kernels(rom.handle) == (
                _lib.ROM_KERNEL_ROWS64 if state == "f64" else _lib.ROM_KERNEL_ROWS)
            assert dt < 0.1
        outs.append(out)
        rom.close()
    # FP64: other summation orders (the parity tests' bar); FP32: the same up to
    # 256 rows, J and y to FP64 rounding above
    for i, tol in enumerate((0.0, 0.0, 1e-12) if state == "f32" else (1e-12,) * 3):
        _compare(outs[0][i], outs[1][i], tol)
    assert np.array_equal(np.isfinite(outs[0][3]), np.isfinite(outs[1][3]))


# Row-split schedule: FP32 resident tiles of one and of two chains per wave and
# streamed rows, BF16 and FP8 operators (states exchanged as BF16 pairs).
@pytest.mark.parametrize("ops,K,M", [("f32", 256, 21), ("f32", 512, 21), ("f32", 1024, 300), ("bf16", 256, 21),
                                     ("bf16", 1024, 70), ("fp8", 512, 40)])
def test_empty_pattern_on_the_row_split_schedule(ops, K, M):
    inst = synth.round_to(synth.make_instance(K, K, M, seed=K + M), "f32")
    rom = _rom(inst, "f32", "rowsplit", ops=ops)
    good, _ = _run(rom, inst, *_states(rom, inst, M, []), 30)
    out, _ = _run(rom, inst, *_states(rom, inst, M, BAD), 30)   # (checks that no wait ran out)
    assert rom.last_schedule == "rowsplit"
    rom.close()
    rest = [m for m in range(M) if m not in BAD]
    for i, (x, z) in enumerate(zip(out, good)):
        x, z = (x.T, z.T) if i == 3 else (x, z)
        assert np.array_equal(x[rest], z[rest])
        assert i == 3 or not np.any(np.all(np.isfinite(x[BAD].reshape(len(BAD), -1)), axis=1))


@pytest.mark.parametrize("state,kv,ks,M,kernel", [("f64", 160, 130, 20, _lib.ROM_KERNEL_ROWS64),
                                                  ("f32", 256, 250, 20, _lib.ROM_KERNEL_ROWS)])
def test_overflowing_run(columns_table, state, kv, ks, M, kernel):
    """A time step far beyond the stability limit: every sample overflows."""
    inst = synth.make_instance(kv, ks, M, seed=9, skew=False)
    columns_table(kv, ks, M)
    N = 400
    outs = []
    for schedule in ("auto", "columns"):
        rom = _rom(inst, state, schedule, dt=1e3 * inst["dt"])
        _run(rom, inst, *_states(rom, inst, M, []), 30)
        out, dt = _run(rom, inst, *_states(rom, inst, M, []), N)
        if schedule == "auto":
            assert _lib.load().rom_debug_kernels(rom.handle) == kernel and dt < 0.1
        outs.append(out)
        rom.close()
    for x, z in zip(*outs):
        assert np.array_equal(np.isfinite(x), np.isfinite(z))
    assert not np.any(np.isfinite(outs[0][0]))


@pytest.mark.parametrize("kv,M", [(64, 1), (40, 5), (64, 64), (256, 130), (100, 700)])
def test_receiver_percentiles_with_nan(kv, M):
    """NaN sorts behind every number in the percentiles (the order of numpy's
    sort), whatever share of the samples they are."""
    from paper_2009_11742_amd import Rom
    inst = synth.round_to(synth.make_instance(kv, kv, M, seed=kv + M, skew=False), "f32")
    rom = Rom(inst["Avs"], inst["Asv"], inst["b"], inst["dt"], state="f32")
    mu = torch.tensor(inst["mu"], dtype=torch.float64, device="cuda")
    C = torch.tensor(np.random.default_rng(kv).standard_normal((3, kv)), dtype=torch.float32, device="cuda")
    for share in (0.02, 0.4, 0.6, 0.97, 1.0):
        nan = np.random.default_rng(1).permutation(M)[:max(1, int(share * M))]
        V, S = rom.zeros(M)
        V += torch.tensor(np.random.default_rng(2).standard_normal((M, kv)), dtype=torch.float32, device="cuda")
        V[torch.tensor(nan, device="cuda"), 0] = float("nan")
        V[torch.tensor([m for m in range(M) if m not in nan][:2], dtype=torch.int64, device="cuda")] *= 1e30
        o = rom.run_receivers(mu, V, S, 2, C)
        rom.check()
        Y, stats = o["Y"].cpu().numpy(), o["stats"].cpu().numpy()
        assert np.all(np.isnan(Y[:, :, nan])) and np.isfinite(Y).sum() == Y[:, :, 0].size * (M - len(nan))
        assert np.all(np.isnan(stats[:, :, :2]))
        srt = np.sort(Y, axis=2)
        for i, p in enumerate((5, 50, 95)):
            assert np.array_equal(stats[:, :, 2 + i], srt[:, :, max(1, -(-p * M // 100)) - 1], equal_nan=True)
    rom.close()
