"""Autotuner of the hop launch parameters (mobius_tune): the chosen parameters
are valid, the operator's results do not change beyond rounding (the
candidates keep the order of the direction sum; only the compiler's choice of
fused multiply-adds may differ between the unrolled variants), and the cache
file is written and re-used."""
import sys

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch_cuda():
    import torch
    assert torch.cuda.is_available(), "GPU tests need an MI355X"
    return torch


def _op(torch, dims=(8, 8, 8, 8), Ls=8, seed=3):
    from paper_1206_5214_amd import inputs, mobius
    rng = np.random.default_rng(seed)
    U = torch.from_numpy(inputs.random_links(dims, 0.5, rng)).cuda()
    psi = torch.from_numpy(inputs.gaussian_spinor(dims, Ls, rng)).cuda()
    return mobius.Operator(dims, Ls, 1.8, 0.01, 1.5, 0.5, U), psi


# rounding-level bound on |after - before| / |before| per storage precision
ROUND = {0: 1e-14, 1: 1e-6, 2: 2e-3}


def test_tune_keeps_results(torch_cuda, monkeypatch):
    from paper_1206_5214_amd import mobius
    torch = torch_cuda
    monkeypatch.delenv("MOBIUS_TUNE_CACHE", raising=False)
    op, psi = _op(torch)
    for prec in (mobius.F64, mobius.F32, mobius.F16):
        e, o = op.pack(psi, prec)
        zero = op.new_field(prec)

        def outputs():
            return [op.unpack(op.dslash(o, 0, prec), zero, prec),
                    op.unpack(zero, op.dslash(e, 1, prec, dag=True), prec),
                    op.unpack(zero, op.dslash(o, 1, prec, op=mobius.OP_SCHUR), prec)]
        before = outputs()
        r = op.tune(prec, reps=3)
        print(f"prec {prec}: {r}", flush=True)
        assert r["prec"] == prec and r["prefetch"] in (0, 1, 2)
        assert r["stage_links"] in (0, 1) and r["xcd_remap"] in (0, 1) and r["nt_links"] in (0, 1)
        assert r["mfma"] in (0, 1)
        assert r["hop_us"] > 0
        after = outputs()
        for a, b in zip(before, after):
            rel = (torch.linalg.vector_norm(a - b) / torch.linalg.vector_norm(b)).item()
            assert rel <= ROUND[prec], (prec, rel)
    op.close()


def test_tune_cache(torch_cuda, monkeypatch, tmp_path):
    from paper_1206_5214_amd import mobius
    torch = torch_cuda
    cache = tmp_path / "tune.txt"
    monkeypatch.setenv("MOBIUS_TUNE_CACHE", str(cache))
    op, psi = _op(torch, dims=(8, 8, 4, 8), Ls=12)
    r1 = op.tune(mobius.F32, reps=3)
    text = cache.read_text()
    assert text.count("\n") == 1 and "Ls12" in text and "prec1" in text
    op.close()
    op2, _ = _op(torch, dims=(8, 8, 4, 8), Ls=12, seed=4)
    r2 = op2.tune(mobius.F32, reps=3)
    assert r2 == r1                       # taken from the cache, not re-timed
    assert cache.read_text() == text      # nothing appended
    sol, info, rc = op2.solve(psi, tol=1e-10, inner_prec=mobius.F32)
    assert rc == mobius.OK and info[0].true_resid <= 1e-10
    op2.close()


def test_tune_cache_of_other_kernels_is_not_used(torch_cuda, monkeypatch, tmp_path):
    """Lines that an older library measured on its own kernels (another version in
    the key, or no split flag at the end) are timed again, and the new line used."""
    from paper_1206_5214_amd import mobius
    torch = torch_cuda
    cache = tmp_path / "tune.txt"
    monkeypatch.setenv("MOBIUS_TUNE_CACHE", str(cache))
    op, _ = _op(torch, dims=(4, 4, 4, 8), Ls=8)
    op.tune(mobius.F64, reps=3)
    key, values = cache.read_text().strip().split(" | ")
    words = values.split()
    words[5] = "123456.5"  # the hop's time
    old = [key.rsplit(" ", 1)[0] + " v2 | " + " ".join(words[:6]), key + " | " + " ".join(words[:6])]
    for line in old:
        cache.write_text(line + "\n")
        r = op.tune(mobius.F64, reps=3)
        lines = cache.read_text().splitlines()
        assert r["hop_us"] != 123456.5 and len(lines) == 2 and lines[0] == line
        assert op.tune(mobius.F64, reps=3) == r and len(cache.read_text().splitlines()) == 2
    op.close()


@pytest.mark.parametrize("prec", [0, 1, 2], ids=["f64", "f32", "f16"])
def test_tuned_choice_survives_the_round_trip(torch_cuda, monkeypatch, prec):
    """What tune reports, handed to another operator's set_tuning, launches the same
    hops: the split form and the depth by kernel included.  set_tuning alone selects
    the loop, at one depth."""
    from paper_1206_5214_amd import mobius
    torch = torch_cuda
    monkeypatch.delenv("MOBIUS_TUNE_CACHE", raising=False)
    op, psi = _op(torch, dims=(4, 4, 4, 8), Ls=8)
    op2, _ = _op(torch, dims=(4, 4, 4, 8), Ls=8)
    assert op.hop_flags(prec) == mobius.HOP_SPLIT | mobius.HOP_DEPTH_BY_KERNEL  # untuned, 8 site blocks
    r = op.tune(prec, reps=3)
    _, o = op.pack(psi, prec)
    for split in (0, 1):
        for by_kernel in (0, 1):
            # the four choices a tuner can make, the one it made among them
            r.update(split=split, depth_by_kernel=by_kernel)
            for q in (op, op2):
                q.set_tuning(**{k: v for k, v in r.items() if k != "hop_us"})
            want = (mobius.HOP_SPLIT if split else 0) | (mobius.HOP_DEPTH_BY_KERNEL if by_kernel else 0)
            assert op.hop_flags(prec) == op2.hop_flags(prec) == want
            # 100 right-hand sides of 8 site blocks are past every precision's threshold
            assert not op.hop_flags(prec, 100) & mobius.HOP_SPLIT
            assert torch.equal(op.dslash(o, 1, prec, op=mobius.OP_SCHUR), op2.dslash(o, 1, prec, op=mobius.OP_SCHUR))
    op.set_tuning(prec, 2, 1, 1, 0)
    assert op.hop_flags(prec) == 0
    for flags in (4, 8, -1):
        assert mobius.lib().mobius_set_hop_flags(op._h, prec, flags) == -22
    assert mobius.lib().mobius_hop_flags(op._h, prec, 0) == -22 and mobius.lib().mobius_hop_flags(op._h, 7, 1) == -22
    assert op.hop_flags(prec) == 0
    op.close()
    op2.close()


@pytest.mark.parametrize("env,split", [({"MOBIUS_XCD_REMAP": "1", "MOBIUS_STAGE_LINKS": "1"}, True),
                                       ({"MOBIUS_XCD_REMAP": "0"}, True), ({"MOBIUS_STAGE_LINKS": "0"}, False),
                                       ({"MOBIUS_PREFETCH": "1"}, False)])
def test_environment_selects_the_loop_only_for_another_variant(torch_cuda, env, split):
    """The process defaults are read once, hence the child process: a hop variable at
    its default value, or the block order, leaves small lattices their split form."""
    import os
    import subprocess
    code = ("import numpy as np, torch; from paper_1206_5214_amd import inputs, mobius; "
            "U = torch.from_numpy(inputs.unit_links((4, 4, 4, 4))).cuda(); "
            "op = mobius.Operator((4, 4, 4, 4), 8, 1.8, 0.1, 1.5, 0.5, U); print('flags', op.hop_flags(0))")
    out = subprocess.run([sys.executable, "-c", code], env={**os.environ, **env}, capture_output=True, text=True,
                         timeout=100, cwd=os.path.dirname(os.path.dirname(os.path.abspath(__file__))))
    assert out.returncode == 0, out.stderr
    flags = int(out.stdout.split("flags")[1])
    from paper_1206_5214_amd import mobius
    assert bool(flags & mobius.HOP_SPLIT) == split


def test_tune_rejects_bad_precision(torch_cuda):
    from paper_1206_5214_amd import mobius
    torch = torch_cuda
    op, _ = _op(torch, dims=(4, 4, 4, 4))
    with pytest.raises(mobius.MobiusError):
        op.tune(7)
    op.close()


LAUNCH_VARIANTS = ([(pf, st, rm, nt, 0) for pf in (0, 1, 2) for st in (0, 1) for rm in (0, 1) for nt in (0, 1)]
                   + [(2, 1, rm, nt, 1) for rm in (0, 1) for nt in (0, 1)])


@pytest.mark.parametrize("prec", [0, 1, 2], ids=["f64", "f32", "f16"])
def test_every_launch_variant_vs_oracle(torch_cuda, orc, prec):
    """Each of the 28 candidates the tuner may pick (the last four: the FP16
    matrix-core colour multiply, the launch parameters alone elsewhere), set
    explicitly, gives the hop blocks (forward and adjoint, both parities) and
    the Schur operator within the storage precision's tolerance of the FP64
    oracle."""
    from oracle import Params
    from paper_1206_5214_amd import inputs, mobius
    torch = torch_cuda
    tol = {0: 1e-12, 1: 2e-5, 2: 4e-3}[prec]
    dims, Ls = (6, 4, 2, 4), 12
    p = Params(dims, Ls, 1.8, 0.05, 1.75, 0.75)
    rng = np.random.default_rng(21)
    U = inputs.random_links(dims, 0.6, rng)
    psi = inputs.gaussian_spinor(dims, Ls, rng)
    want = [orc.hop(p, U, psi, q, dag=d) for q in (0, 1) for d in (False, True)]
    want_schur = orc.schur(p, U, orc.restrict(p, psi, 1))
    op = mobius.Operator(dims, Ls, 1.8, 0.05, 1.75, 0.75, torch.from_numpy(U).cuda())
    e, o = op.pack(torch.from_numpy(psi).cuda(), prec)
    zero = op.new_field(prec)
    for v in LAUNCH_VARIANTS:
        op.set_tuning(prec, *v)
        got = []
        for q in (0, 1):
            for d in (False, True):
                src = o if q == 0 else e
                out = op.dslash(src, q, prec, dag=d)
                got.append(op.unpack(out, zero, prec) if q == 0 else op.unpack(zero, out, prec))
        for g, w in zip(got, want):
            g = g.cpu().numpy()
            assert np.linalg.norm(g - w) <= tol * np.linalg.norm(w), (v, prec)
        s = op.unpack(zero, op.dslash(o, 1, prec, op=mobius.OP_SCHUR), prec).cpu().numpy()
        assert np.linalg.norm(s - want_schur) <= tol * np.linalg.norm(want_schur), (v, prec)
    with pytest.raises(mobius.MobiusError):
        op.set_tuning(prec, 3, 0, 0, 0)
    with pytest.raises(mobius.MobiusError):
        op.set_tuning(prec, 2, 1, 0, 0, 2)
    op.close()


def test_tune_brick_and_explicit_site_order(torch_cuda, monkeypatch):
    """The layout tuner (mobius_tune_brick) times candidate site-order bricks,
    the automatic one first, and returns one of them; an operator created with
    an explicit brick, including one that does not divide the lattice, gives
    per site exactly the hops of the automatic order in every precision (the
    order only moves sites between workgroups) and solves to the same accuracy."""
    from paper_1206_5214_amd import inputs, mobius
    torch = torch_cuda
    monkeypatch.delenv("MOBIUS_TUNE_CACHE", raising=False)
    dims, Ls = (8, 8, 4, 4), 8
    rng = np.random.default_rng(21)
    U = torch.from_numpy(inputs.random_links(dims, 0.5, rng)).cuda()
    psi = torch.from_numpy(inputs.gaussian_spinor(dims, Ls, rng)).cuda()
    args = (dims, Ls, 1.8, 0.05, 1.5, 0.5)
    brick, us, trials = mobius.tune_brick(*args, U, prec=mobius.F16, reps=2)
    print(f"brick {brick} {us:.1f} us; trials {trials}", flush=True)
    assert 2 <= len(trials) <= 12 and all(t[1] > 0 for t in trials)
    assert brick in [t[0] for t in trials]
    for b, _ in trials[1:]:
        assert all(1 <= b[k] <= dims[k] and dims[k] % b[k] == 0 for k in range(3))
    auto_us = trials[0][1]
    assert (brick == trials[0][0] and us == auto_us) or us < 0.97 * auto_us
    op0 = mobius.Operator(*args, U)
    for b in ((2, 2, 2), (4, 8, 2), (6, 8, 4), brick):
        op1 = mobius.Operator(*args, U, brick=b)
        for prec in (mobius.F64, mobius.F32, mobius.F16):
            outs = []
            for op in (op0, op1):
                e, o = op.pack(psi, prec)
                zero = op.new_field(prec)
                outs.append([op.unpack(op.dslash(o, 0, prec), zero, prec),
                             op.unpack(zero, op.dslash(e, 1, prec, dag=True), prec)])
            for a, c in zip(*outs):
                assert torch.equal(a, c), (b, prec)
        sol, info, rc = op1.solve(psi, tol=1e-10, inner_prec=mobius.F16)
        assert rc == mobius.OK and info[0].true_resid <= 1e-10
        op1.close()
    op0.close()
