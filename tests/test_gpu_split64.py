"""FP64 row-split schedule (FP64 states, max(Kv_pad, Ks_pad) in 128 .. 512
between the resident and the panel kernels): groups of 16 samples over the
workgroups of one XCD, rows exchanged through polled slots.

Against the FP64 oracle at the FP64 bar (1e-12 per-sample relative l2; J and
the probe trace relative) at the smallest and largest padded sizes, Kv !=
Ks both ways, a part-filled last group, and more groups than fit at once
(rounds); bitwise independence of a sample from its companions and from the
number of rounds' predecessors; runs of one context on two streams; the
host-forced time-out.
"""
import numpy as np
import pytest

import oracle
import synth
from paper_2009_11742_amd import _lib

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu
BAR64 = 1e-12


def _rel(X, R):
    return float(np.max(np.linalg.norm(X - R, axis=0) / np.linalg.norm(R, axis=0)))


def _rom(inst, **kw):
    from paper_2009_11742_amd import Rom
    return Rom(inst["Avs"], inst["Asv"], inst["b"], inst["dt"], state="f64", **kw)


def _run(rom, inst, mu_np, N, n0=0):
    M = len(mu_np)
    mu = torch.tensor(mu_np, dtype=torch.float64, device="cuda")
    V, S = rom.zeros(M)
    c = torch.tensor(inst["c"], dtype=torch.float64, device="cuda")
    J = torch.zeros(M, dtype=torch.float64, device="cuda")
    y = torch.zeros((N, M), dtype=torch.float64, device="cuda")
    rom.run_rank2(mu, V, S, N, n0=n0, c=c, J=J, y=y)
    rom.check()
    return [t.cpu().numpy() for t in (V, S, J, y)]


# (128, 128): the smallest; (130, 70), (70, 180): ragged, Kv != Ks; (512, 64)
# and (64, 512): the largest, one field of one tile; (300, 280, 390): 32-row
# tiles; (192, 192, 1100): three rounds of 32-row tiles, last group ragged.
@pytest.mark.parametrize("kv,ks,M,N", [(128, 128, 1, 200), (130, 70, 17, 200), (70, 180, 16, 150),
                                       (512, 64, 5, 100), (64, 512, 33, 100), (300, 280, 390, 60),
                                       (192, 192, 1100, 40)])
def test_split64_parity(kv, ks, M, N):
    inst = synth.make_instance(kv, ks, M, seed=kv + 3 * ks + M, skew=False)
    rom = _rom(inst)
    V, S, J, y = _run(rom, inst, inst["mu"], N, n0=3)
    rom.close()
    cols = np.unique(np.linspace(0, M - 1, 20).astype(int))
    ref = oracle.run_rank2(inst["Avs"], inst["Asv"], inst["b"], inst["dt"], inst["mu"][cols], N, n0=3, c=inst["c"],
                           trace=True)
    e = (_rel(V.T[:, cols], ref["V"]), _rel(S.T[:, cols], ref["S"]),
         float(np.max(np.abs(J[cols] - ref["J"]) / ref["J"])),
         float(np.max(np.abs(y[:, cols] - ref["y"])) / np.max(np.abs(ref["y"]))))
    print("split f64 K=(%d,%d) M=%d N=%d: V %.2e S %.2e J %.2e y %.2e" % ((kv, ks, M, N) + e))
    assert max(e) <= BAR64
    assert np.all(np.isfinite(V)) and np.all(np.isfinite(S))


def test_split64_sample_does_not_depend_on_its_companions():
    """All samples in one round against the same samples among more than fit
    at once: bitwise, for both row tiles."""
    inst = synth.make_instance(192, 150, 900, seed=5, skew=False)
    rom = _rom(inst)
    big = _run(rom, inst, inst["mu"], 50)
    few = _run(rom, inst, inst["mu"][[899, 4, 640]], 50)
    for a, b in zip(big, few):
        if a.shape[0] == 900:
            assert np.allclose(a[[899, 4, 640]], b, rtol=1e-13, atol=1e-13 * np.max(np.abs(a)))
    again = _run(rom, inst, inst["mu"], 50)
    for a, b in zip(big, again):
        assert np.array_equal(a, b)
    perm = np.random.default_rng(1).permutation(900)
    p = _run(rom, inst, inst["mu"][perm], 50)
    assert np.array_equal(p[0], big[0][perm]) and np.array_equal(p[1], big[1][perm])
    assert np.array_equal(p[2], big[2][perm]) and np.array_equal(p[3], big[3][:, perm])
    rom.close()


def test_split64_two_streams_of_one_context():
    """The exchange workspace is the context's: runs enqueued on two streams
    give what they give alone."""
    inst = synth.make_instance(200, 200, 40, seed=6)
    rom = _rom(inst)
    N = 400
    mu = torch.tensor(inst["mu"], dtype=torch.float64, device="cuda")
    ref = _run(rom, inst, inst["mu"], N)
    streams = [torch.cuda.Stream(), torch.cuda.Stream()]
    outs = [rom.zeros(40) for _ in range(4)]
    torch.cuda.synchronize()
    for i, (V, S) in enumerate(outs):
        rom.run_rank2(mu, V, S, N, stream=streams[i % 2])
    torch.cuda.synchronize()
    rom.check()
    for V, S in outs:
        assert np.array_equal(V.cpu().numpy(), ref[0]) and np.array_equal(S.cpu().numpy(), ref[1])
    rom.close()


def test_split64_reports_timeout_and_recovers():
    inst = synth.make_instance(160, 160, 20, seed=7)
    rom = _rom(inst)
    mu = torch.tensor(inst["mu"], dtype=torch.float64, device="cuda")
    ref = _run(rom, inst, inst["mu"], 100)
    lib = _lib.load()
    lib.rom_debug_force_timeout(1)
    try:
        V, S = rom.zeros(20)
        rom.run_rank2(mu, V, S, 50)
        with pytest.raises(_lib.RomError) as ei:
            rom.check()
        assert ei.value.status == _lib.ROM_E_TIMEOUT
    finally:
        lib.rom_debug_force_timeout(0)
    rom.check()
    out = _run(rom, inst, inst["mu"], 100)
    for a, b in zip(out, ref):
        assert np.array_equal(a, b)
    rom.close()


def test_split64_captured_run_stays_on_the_column_blocks():
    inst = synth.make_instance(160, 130, 6, seed=8, skew=False)
    rom, pinned = _rom(inst), _rom(inst, schedule="columns")
    mu = torch.tensor(inst["mu"], dtype=torch.float64, device="cuda")
    V, S = rom.zeros(6)
    s, g = torch.cuda.Stream(), torch.cuda.CUDAGraph()
    torch.cuda.synchronize()
    with torch.cuda.graph(g, stream=s):
        rom.run_rank2(mu, V, S, 60, stream=s)
    Vp, Sp = rom.zeros(6)
    pinned.run_rank2(mu, Vp, Sp, 60)
    for _ in range(3):
        V.zero_(); S.zero_()
        torch.cuda.synchronize()
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(V, Vp) and torch.equal(S, Sp)
        rom.run_rank2(mu, *rom.zeros(6), 5)
        torch.cuda.synchronize()
    rom.close(); pinned.close()


@pytest.mark.parametrize("kv,ks,M,few", [(192, 150, 900, [899, 4, 640]), (128, 128, 600, list(range(250, 290))),
                                         (300, 280, 390, [0, 17, 389]), (64, 512, 140, [139]), (512, 64, 140, [3, 70])])
def test_split64_bits_do_not_depend_on_the_company(kv, ks, M, few):
    """More samples than 16-row tiles hold at once (32-row tiles, (192, 150)
    and (300, 280) in rounds) against some of them alone (16-row tiles)."""
    inst = synth.make_instance(kv, ks, M, seed=kv + M, skew=False)
    rom = _rom(inst)
    big, alone = _run(rom, inst, inst["mu"], 40, n0=2), _run(rom, inst, inst["mu"][few], 40, n0=2)
    rom.close()
    for a, b in zip((big[0][few], big[1][few], big[2][few], big[3][:, few]), alone):
        assert np.array_equal(a, b)


@pytest.mark.parametrize("kv,ks,M", [(128, 128, 3), (130, 70, 17), (300, 280, 40), (64, 512, 33), (512, 64, 5)])
@pytest.mark.parametrize("cut", [1, 2, 4])
def test_split64_run_cut_into_few_steps(kv, ks, M, cut):
    """Runs of a few steps, launched per half-step, give the states and the
    probe trace of one run, bit for bit; J to the order of its sum."""
    inst = synth.make_instance(kv, ks, M, seed=kv + M, skew=False)
    rom = _rom(inst)
    N = 12
    V, S, J, y = _run(rom, inst, inst["mu"], N, n0=4)
    mu = torch.tensor(inst["mu"], dtype=torch.float64, device="cuda")
    c = torch.tensor(inst["c"], dtype=torch.float64, device="cuda")
    (V2, S2), (V3, S3) = rom.zeros(M), rom.zeros(M)
    J2 = torch.zeros(M, dtype=torch.float64, device="cuda")
    y2 = torch.zeros((N, M), dtype=torch.float64, device="cuda")
    for k in range(0, N, cut):
        rom.run_rank2(mu, V2, S2, cut, n0=4 + k, c=c, J=J2, y=y2[k:k + cut])
        rom.run_rank2(mu, V3, S3, cut, n0=4 + k)
    rom.check()
    rom.close()
    for a, b in ((V, V2), (S, S2), (y, y2), (V, V3), (S, S3)):
        assert np.array_equal(a, b.cpu().numpy())
    assert np.max(np.abs(J2.cpu().numpy() - J) / J) <= 1e-14
