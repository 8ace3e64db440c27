"""Which kernels a call launches (rom_debug_kernels), so that the tests that
compare kernels with each other compare what they mean to: the small models'
kernels, the resident row-split kernels with the column blocks' sums, the FP64
row-split kernels, and the column blocks where a context pins them.
"""
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


def _launched(kv, ks, M, state, schedule="auto", call="run", N=200):
    from paper_2009_11742_amd import Rom
    inst = synth.make_instance(kv, ks, M, seed=1, skew=False)
    rom = Rom(inst["Avs"], inst["Asv"], inst["b"], inst["dt"], state=state, schedule=schedule)
    mu = torch.tensor(inst["mu"], dtype=torch.float64, device="cuda")
    V, S = rom.zeros(M)
    if call == "run":
        rom.run_rank2(mu, V, S, N)
    else:
        rom.run_receivers(mu, V, S, N, torch.ones((2, kv), dtype=torch.float32, device="cuda"))
    rom.check()
    k = _lib.load().rom_debug_kernels(rom.handle)
    rom.close()
    return k


CHAINS = [(1, 1, 1), (64, 63, 257), (113, 128, 1001), (192, 128, 40), (131, 190, 300), (256, 64, 260), (70, 193, 300),
          # 192 padded rows: few or many samples, or more than 160 rows
          (150, 130, 200), (150, 130, 385), (192, 130, 1), (130, 192, 17), (192, 192, 700)]
ROWS = [(150, 130, 300), (160, 129, 384), (256, 192, 20), (192, 256, 300), (256, 200, 128), (250, 256, 500), (256, 256, 512), (300, 280, 33),
        (64, 512, 16), (512, 500, 129), (512, 512, 500), (700, 600, 128), (600, 768, 250),
        (1000, 1024, 100), (1024, 900, 256)]
# No tile that holds all their groups is faster.
BLOCKS = [(512, 40, 250), (256, 256, 513), (256, 256, 700), (200, 256, 1024), (256, 256, 1025)]


@pytest.mark.parametrize("call", ["run", "receivers"])
@pytest.mark.parametrize("kv,ks,M,kernel", [s + (_lib.ROM_KERNEL_CHAINS,) for s in CHAINS] +
                         [s + (_lib.ROM_KERNEL_ROWS,) for s in ROWS] + [s + (_lib.ROM_KERNEL_COLUMNS,) for s in BLOCKS])
def test_column_block_runs(columns_table, kv, ks, M, kernel, call):
    if call == "receivers":
        M = min(M, 1024)        # their limit
    columns_table(kv, ks, M)
    assert _launched(kv, ks, M, "f32", call=call) == kernel
    assert _launched(kv, ks, M, "f32", schedule="columns", call=call) == _lib.ROM_KERNEL_COLUMNS


@pytest.mark.parametrize("call", ["run", "receivers"])
@pytest.mark.parametrize("kv,ks,M,short,long", [(256, 256, 64, 4, 30), (300, 280, 100, 1, 20), (500, 1000, 100, 0, 4)])
def test_short_runs_stay_on_the_column_blocks(columns_table, kv, ks, M, short, long, call):
    """A row-split call costs about 20 us beside its steps."""
    columns_table(kv, ks, M)
    assert _launched(kv, ks, M, "f32", call=call, N=short) == (_lib.ROM_KERNEL_COLUMNS if short else 0)
    assert _launched(kv, ks, M, "f32", call=call, N=long) == _lib.ROM_KERNEL_ROWS


@pytest.mark.parametrize("M", [600, 1500, 2048, 4096])
def test_tuner_takes_the_fastest_where_columns_run_as_timed(M):
    """K = 256: where a column-block run takes the column-block kernels, the
    tuner may choose any schedule, row-split too."""
    from paper_2009_11742_amd import Rom, tuning
    tuning.load_default()
    saved = tuning.entries()
    inst = synth.make_instance(256, 256, M, seed=1, skew=False)
    rom = Rom(inst["Avs"], inst["Asv"], inst["b"], inst["dt"], state="f32")
    try:
        tuning.clear()
        V, S = rom.zeros(M)
        rom.run_rank2(torch.tensor(inst["mu"], dtype=torch.float64, device="cuda"), V, S, 20)
        times = {k: t for k, t in rom.schedule_times(M).items() if t is not None}
        assert times[rom.last_schedule] == min(times.values()), (rom.last_schedule, times)
    finally:
        rom.close()
        tuning.clear()
        for e in saved:
            tuning.put(e["kv_pad"], e["ks_pad"], e["m_pad"], e["op"], e["schedule"], e["us"])


@pytest.mark.parametrize("kv,ks,M", [(128, 128, 1), (130, 70, 17), (70, 180, 16), (512, 64, 5), (64, 512, 33),
                                     (300, 280, 390), (192, 192, 1100)])
def test_fp64_runs(kv, ks, M):
    assert _launched(kv, ks, M, "f64") == _lib.ROM_KERNEL_ROWS64
    assert _launched(kv, ks, M, "f64", schedule="columns") == _lib.ROM_KERNEL_VALU64


@pytest.mark.parametrize("kv,ks,M,skew", [(256, 256, 20, True), (250, 250, 40, False), (256, 500, 30, False)])
def test_adjoint_of_column_sweeps_does_not_wait(kv, ks, M, skew):
    """Adjoints whose forward sweep is not on the row-split schedule enqueue
    their sweeps (column blocks) and return: here behind another run of about
    0.1 s on the same stream."""
    from paper_2009_11742_amd import Rom
    inst = synth.make_instance(kv, ks, M, seed=1, skew=skew)
    rom = Rom(inst["Avs"], inst["Asv"], inst["b"], inst["dt"], state="f32")
    mu = torch.tensor(inst["mu"], dtype=torch.float64, device="cuda")
    c = torch.tensor(inst["c"], dtype=torch.float32, device="cuda")
    rom.adjoint(mu, 40, c)          # tunes the shape, allocates
    assert rom.last_schedule != "rowsplit"
    big = synth.make_instance(1024, 1024, 4, seed=2)
    long = Rom(big["Avs"], big["Asv"], big["b"], big["dt"], state="f32", schedule="columns")
    V, S = long.zeros(4)
    bmu = torch.tensor(big["mu"], dtype=torch.float64, device="cuda")
    long.run_rank2(bmu, V, S, 1)
    torch.cuda.synchronize()
    long.run_rank2(bmu, V, S, 1500)
    out = rom.adjoint(mu, 40, c)
    assert not torch.cuda.current_stream().query()
    torch.cuda.synchronize()
    assert _lib.load().rom_debug_kernels(rom.handle) & _lib.ROM_KERNEL_COLUMNS
    again = rom.adjoint(mu, 40, c)
    for k in out:
        assert torch.equal(out[k], again[k])
    rom.close(); long.close()


@pytest.mark.parametrize("ops", ["bf16", "fp8"])
@pytest.mark.parametrize("K,M", [(128, 1), (91, 142), (128, 600)])
def test_tuner_keeps_small_low_precision_models_on_column_blocks(ops, K, M):
    from paper_2009_11742_amd import Rom, tuning
    tuning.load_default()
    saved = tuning.entries()
    inst = synth.make_instance(K, K, M, seed=1)
    outs = []
    try:
        tuning.clear()
        for schedule in ("auto", "columns"):
            rom = Rom(inst["Avs"], inst["Asv"], inst["b"], inst["dt"], state="f32", ops=ops, schedule=schedule)
            V, S = rom.zeros(M)
            rom.run_rank2(torch.tensor(inst["mu"], dtype=torch.float64, device="cuda"), V, S, 30)
            assert rom.last_schedule == "columns"
            outs.append((V, S))
            rom.close()
    finally:
        tuning.clear()
        for e in saved:
            tuning.put(e["kv_pad"], e["ks_pad"], e["m_pad"], e["op"], e["schedule"], e["us"])
    assert torch.equal(outs[0][0], outs[1][0]) and torch.equal(outs[0][1], outs[1][1])
