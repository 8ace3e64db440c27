"""Runs that take row-split kernels without having been asked for that schedule
(FP32 column-block runs, receivers, forward sweeps of adjoints, FP64 runs
between the resident and the panel sizes) do not fail where a wait of those kernels runs
out: the samples are left as they were and done by the column blocks behind.

The time-out is forced from the host; the results must then be those of a
context pinned to the column blocks, bit for bit, and (FP32) nothing may be
reported.  rom_debug_kernels shows that the row-split kernels were launched.
"""
import numpy as np
import pytest

import synth
from paper_2009_11742_amd import _lib

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu


@pytest.fixture
def forced():
    lib = _lib.load()
    lib.rom_debug_force_timeout(1)
    try:
        yield
    finally:
        lib.rom_debug_force_timeout(0)


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


def _rom(inst, state, schedule="auto"):
    from paper_2009_11742_amd import Rom
    return Rom(inst["Avs"], inst["Asv"], inst["b"], inst["dt"], state=state, schedule=schedule)


def _kernels(rom):
    return _lib.load().rom_debug_kernels(rom.handle)


def _inst(kv, ks, M):
    return synth.round_to(synth.make_instance(kv, ks, M, seed=kv + 3 * ks + M, skew=False), "f32")


def _run(rom, inst, M, N):
    t = rom.torch_dtype
    mu = torch.tensor(inst["mu"][:M], dtype=torch.float64, device="cuda")
    V, S = rom.zeros(M)
    V += 1e-3 * torch.tensor(inst["b"], dtype=t, device="cuda")
    c = torch.tensor(inst["c"], dtype=t, device="cuda")
    J = torch.ones(M, dtype=torch.float64, device="cuda")
    y = torch.zeros((N, M), dtype=torch.float64, device="cuda")
    rom.run_rank2(mu, V, S, N, n0=5, c=c, J=J, y=y)
    return [V, S, J, y]


@pytest.mark.parametrize("kv,ks,M", [(256, 256, 70), (300, 280, 33), (64, 512, 20), (500, 1000, 40), (700, 600, 128)])
def test_column_runs_are_repeated(columns_table, forced, kv, ks, M):
    inst = _inst(kv, ks, M)
    columns_table(kv, ks, M)
    outs = []
    for sched in ("auto", "columns"):
        rom = _rom(inst, "f32", sched)
        outs.append(_run(rom, inst, M, 30))
        rom.check()
        assert _kernels(rom) == (_lib.ROM_KERNEL_ROWS if sched == "auto" else _lib.ROM_KERNEL_COLUMNS)
        rom.close()
    for a, b in zip(*outs):
        assert torch.equal(a, b)


@pytest.mark.parametrize("kv,ks,M,N", [(256, 200, 64, 40), (300, 340, 7, 30)])
def test_receiver_runs_are_repeated(forced, kv, ks, M, N):
    inst = _inst(kv, ks, M)
    mu = torch.tensor(inst["mu"], dtype=torch.float64, device="cuda")
    C = torch.tensor(np.random.default_rng(1).standard_normal((3, kv)), dtype=torch.float32, device="cuda")
    outs = []
    for sched in ("auto", "columns"):
        rom = _rom(inst, "f32", sched)
        V, S = rom.zeros(M)
        o = rom.run_receivers(mu, V, S, N, C)
        rom.check()
        assert _kernels(rom) == (_lib.ROM_KERNEL_ROWS if sched == "auto" else _lib.ROM_KERNEL_COLUMNS)
        outs.append([V, S, o["Y"], o["stats"]])
        rom.close()
    for a, b in zip(*outs):
        assert torch.equal(a, b)


# The forward sweep (the other sweeps are on the column blocks).
@pytest.mark.parametrize("kv,ks,M,stride", [(450, 300, 130, 0), (450, 300, 130, -1), (256, 256, 40, -1),
                                            (250, 256, 40, 50)])
def test_adjoints_are_repeated(columns_table, forced, kv, ks, M, stride):
    inst = _inst(kv, ks, M)
    columns_table(kv, ks, M)
    mu = torch.tensor(inst["mu"], dtype=torch.float64, device="cuda")
    c = torch.tensor(inst["c"], dtype=torch.float32, device="cuda")
    outs = []
    for sched in ("auto", "columns"):
        rom = _rom(inst, "f32", sched)
        outs.append(rom.adjoint(mu, 50, c, stride=stride))
        rom.check()
        assert bool(_kernels(rom) & _lib.ROM_KERNEL_ROWS) == (sched == "auto")
        rom.close()
    for k in outs[0]:
        assert torch.equal(outs[0][k], outs[1][k]), k


@pytest.mark.parametrize("kv,ks,M", [(160, 130, 20), (300, 280, 128), (192, 192, 1100)])
def test_fp64_runs_are_repeated(forced, kv, ks, M):
    inst = synth.make_instance(kv, ks, M, seed=kv + M, skew=False)
    rom = _rom(inst, "f64")
    a = _run(rom, inst, M, 12)
    assert _kernels(rom) == _lib.ROM_KERNEL_ROWS64
    with pytest.raises(_lib.RomError) as ei:      # (recorded because it was forced)
        rom.check()
    assert ei.value.status == _lib.ROM_E_TIMEOUT
    rom.check()
    pinned = _rom(inst, "f64", "columns")
    b = _run(pinned, inst, M, 12)
    assert _kernels(pinned) == _lib.ROM_KERNEL_VALU64
    rom.close(); pinned.close()
    for x, y in zip(a, b):
        assert torch.equal(x, y)


@pytest.mark.parametrize("state", ["f64", "f32"])
def test_runs_on_two_threads_default_streams(columns_table, state):
    """hipStreamPerThread is one handle for another stream in each thread: the
    second run, which uses the context's exchange workspace too, waits for the
    first."""
    import ctypes as C
    import threading
    kv, ks, M, N = (200, 180, 40, 3000) if state == "f64" else (256, 250, 40, 4000)
    columns_table(kv, ks, M)
    inst = synth.make_instance(kv, ks, M, seed=3, skew=False)
    rom = _rom(inst, state)
    lib, handle = _lib.load(), rom.handle
    mu = torch.tensor(inst["mu"], dtype=torch.float64, device="cuda")
    ref = rom.zeros(M)
    rom.run_rank2(mu, *ref, N)
    assert _kernels(rom) == (_lib.ROM_KERNEL_ROWS64 if state == "f64" else _lib.ROM_KERNEL_ROWS)
    outs = [rom.zeros(M) for _ in range(2)]
    torch.cuda.synchronize()
    errors, first, second, end = [], threading.Event(), threading.Event(), threading.Event()

    def run(V, S):
        p = lambda t: C.c_void_p(t.data_ptr())
        errors.append(lib.rom_run_rank2(handle, M, p(mu), 0, N, p(V), p(S), None, None, None, C.c_void_p(2)))

    def one():
        run(*outs[0])
        first.set()
        end.wait(60)            # (its stream ends with the thread)

    def two():
        first.wait(60)
        run(*outs[1])
        second.set()
        end.wait(60)

    threads = [threading.Thread(target=f) for f in (one, two)]
    for t in threads:
        t.start()
    second.wait(60)
    torch.cuda.synchronize()
    end.set()
    for t in threads:
        t.join()
    rom.check()
    assert errors == [0, 0]
    for V, S in outs:
        assert torch.equal(V, ref[0]) and torch.equal(S, ref[1])
    rom.close()


def test_row_split_runs_of_several_contexts_take_turns():
    """Kernels whose workgroups wait for each other, from three threads on
    streams of their own (FP64, FP32 column-block and row-split runs): each
    gives what it gives alone, and no wait runs out (which takes about half a
    second)."""
    import threading
    import time
    jobs = []
    for state, kv, ks, M, schedule in (("f64", 300, 280, 128, "auto"), ("f32", 300, 280, 100, "auto"),
                                       ("f32", 512, 512, 100, "rowsplit")):
        inst = synth.make_instance(kv, ks, M, seed=4, skew=kv == ks)
        rom = _rom(inst, state, schedule)
        mu = torch.tensor(inst["mu"], dtype=torch.float64, device="cuda")
        ref = rom.zeros(M)
        rom.run_rank2(mu, *ref, 200)
        outs = [rom.zeros(M) for _ in range(15)]
        jobs.append((rom, mu, ref, outs, torch.cuda.Stream()))
    assert [_kernels(j[0]) for j in jobs] == [_lib.ROM_KERNEL_ROWS64, _lib.ROM_KERNEL_ROWS, 0]
    torch.cuda.synchronize()

    def run(rom, mu, ref, outs, stream):
        for V, S in outs:
            rom.run_rank2(mu, V, S, 200, stream=stream)

    threads = [threading.Thread(target=run, args=j) for j in jobs]
    t0 = time.perf_counter()
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    torch.cuda.synchronize()
    assert time.perf_counter() - t0 < 0.3
    for rom, mu, ref, outs, stream in jobs:
        rom.check()
        for V, S in outs:
            assert torch.equal(V, ref[0]) and torch.equal(S, ref[1])
        rom.close()


# (f64, 192, 192): 40 slots of one or two rounds each, 32-row tiles
@pytest.mark.parametrize("state,kv,ks,M,nc,slots", [
    ("f64", 160, 130, 100, 16, 7), ("f64", 192, 192, 1100, 16, 40), ("f32", 256, 256, 250, 16, 16),
    ("f32", 320, 300, 600, 32, 19), ("f32", 700, 600, 120, 16, 8)])
def test_some_groups_are_repeated(columns_table, state, kv, ks, M, nc, slots):
    """Every other group (FP64: slot of groups) given up: its samples are the
    column blocks', the others the row-split kernels' own."""
    inst = _inst(kv, ks, M)
    columns_table(kv, ks, M)
    lib = _lib.load()
    rom, pinned = _rom(inst, state), _rom(inst, state, "columns")
    own, blocks = _run(rom, inst, M, 30), _run(pinned, inst, M, 30)
    lib.rom_debug_force_timeout(2)
    try:
        got = _run(rom, inst, M, 30)
    finally:
        lib.rom_debug_force_timeout(0)
    rom.check()
    rom.close(); pinned.close()
    odd = torch.tensor(np.arange(M) // nc % slots % 2 == 1, device="cuda")
    for i, (g, o, b) in enumerate(zip(got, own, blocks)):
        g, o, b = (x.T if i == 3 else x.reshape(M, -1) for x in (g, o, b))
        assert torch.equal(g[odd], b[odd]) and torch.equal(g[~odd], o[~odd])
    if state == "f64":          # (the two differ in their last bits)
        assert not torch.equal(own[0][odd], blocks[0][odd])
