"""Kernels at the sizes where their tiling can go wrong: partial last
workgroups, idle lanes, several right-hand sides (GPU)."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch_cuda():
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    return torch


def _setup(torch, dims, Ls, nrhs, seed=3, **kw):
    from paper_1206_5214_amd import inputs, mobius
    rng = np.random.default_rng(seed)
    U = inputs.random_links(dims, 0.4, rng)
    eta = inputs.gaussian_spinor(dims, Ls, rng, nrhs if nrhs > 1 else None)
    op = mobius.Operator(dims, Ls, 1.8, 0.05, 1.5, 0.5, torch.from_numpy(U).cuda(), **kw)
    return mobius, op, torch.from_numpy(eta).cuda()


# 5d sites per parity below, at and past one workgroup's 64, and one site per
# wavefront (Ls > 32)
@pytest.mark.parametrize("dims,Ls", [((2, 2, 2, 2), 2), ((2, 2, 2, 4), 4), ((4, 2, 2, 6), 5),
                                     ((6, 4, 2, 4), 33), ((4, 4, 4, 4), 8)])
@pytest.mark.parametrize("nrhs", [1, 3])
def test_pack_unpack_exact(torch_cuda, dims, Ls, nrhs):
    """FP64 is a permutation, FP32 one rounding, FP16 within one binary16 step
    of the site's largest component (half a step of rounding and the norm's)."""
    torch = torch_cuda
    mobius, op, eta = _setup(torch, dims, Ls, nrhs)
    for prec in (mobius.F64, mobius.F32, mobius.F16):
        even, odd = op.pack(eta, prec, nrhs)
        got = op.unpack(even, odd, prec, nrhs)
        assert got.shape == eta.shape
        if prec == mobius.F64:
            assert torch.equal(got, eta)
        elif prec == mobius.F32:
            assert torch.equal(got, eta.to(torch.complex64).to(torch.complex128))
        else:
            v = torch.view_as_real(eta)
            top = v.abs().amax(dim=(-3, -2, -1), keepdim=True)
            assert ((torch.view_as_real(got) - v).abs() <= 2.0**-11 * top).all()
        if nrhs > 1:  # each right-hand side as by itself
            fb = op.field_bytes(prec)
            for r in range(nrhs):
                e1, o1 = op.pack(eta[r].contiguous(), prec)
                assert torch.equal(e1, even[r * fb:(r + 1) * fb])
                assert torch.equal(o1, odd[r * fb:(r + 1) * fb])
    op.close()


# the s-direction operators on fields in records: fewer sites than one wavefront's,
# partial last wavefronts and workgroups, moved as one stretch (Ls = 4, 12, 20, 28)
# and read directly (Ls = 8, and 36 with one site per wavefront)
@pytest.mark.parametrize("dims,Ls", [((2, 2, 2, 2), 4), ((4, 4, 4, 6), 4), ((4, 2, 2, 6), 12), ((6, 4, 2, 4), 20),
                                     ((2, 2, 2, 6), 28), ((2, 2, 2, 6), 8), ((4, 4, 2, 2), 36)])
@pytest.mark.parametrize("prec,tol", [(0, 1e-12), (1, 2e-5)], ids=["f64", "f32"])
def test_s_direction_operators_vs_oracle(torch_cuda, orc, dims, Ls, prec, tol):
    """I, I^+, I^-1 and I^-+ of two right-hand sides against the FP64 oracle (a
    lane's sums have Ls terms of order one: the hop's tolerances hold)."""
    from oracle import Params
    from paper_1206_5214_amd import inputs
    from parity import check
    torch = torch_cuda
    mobius, op, eta = _setup(torch, dims, Ls, 2)
    p, psi, U = Params(dims, Ls, 1.8, 0.05, 1.5, 0.5), eta.cpu().numpy(), inputs.unit_links(dims)  # (no links enter)
    even, odd = op.pack(eta, prec, 2)
    for dag in (False, True):
        m5 = [op.dslash(x, q, prec, op=mobius.OP_M5, dag=dag, nrhs=2) for q, x in enumerate((even, odd))]
        inv = [op.m5inv(x, prec, dag=dag, nrhs=2) for x in (even, odd)]
        for halves, ref in ((m5, lambda v: orc.m5(p, U, v, dag=dag)), (inv, lambda v: orc.m5inv(p, v, dag=dag))):
            got = op.unpack(*halves, prec, 2).cpu().numpy()
            for r in range(2):
                check(got[r], ref(psi[r]), tol, (dims, Ls, dag, r))
    op.close()


# the same on fields past the L2s, which move as one stretch in both types (Ls = 4:
# 32 MB, longer Ls: 32 MB in FP32, 96 MB in FP64), with a partial last wavefront
@pytest.mark.parametrize("dims,Ls", [((18, 14, 14, 50), 4), ((18, 14, 14, 26), 12), ((14, 14, 10, 34), 20)])
def test_s_direction_operators_on_large_fields(torch_cuda, orc, dims, Ls):
    """I and I^-1 and their adjoints in both types against the FP64 oracle, with the
    tolerances of the small lattices (a lane's sums have the same Ls terms)."""
    from oracle import Params
    from paper_1206_5214_amd import inputs
    from parity import check
    torch = torch_cuda
    mobius, op, eta = _setup(torch, dims, Ls, 1)
    assert op.field_bytes(mobius.F32) >= 32 << 20 and op.field_bytes(mobius.F64) >= (32 if Ls == 4 else 96) << 20
    p, psi, U = Params(dims, Ls, 1.8, 0.05, 1.5, 0.5), eta.cpu().numpy(), inputs.unit_links(dims)  # (no links enter)
    for dag in (False, True):
        m5, inv = orc.m5(p, U, psi, dag=dag), orc.m5inv(p, psi, dag=dag)
        for prec, tol in ((mobius.F64, 1e-12), (mobius.F32, 2e-5)):
            halves = op.pack(eta, prec)
            for ref, got in ((m5, [op.dslash(x, q, prec, op=mobius.OP_M5, dag=dag) for q, x in enumerate(halves)]),
                             (inv, [op.m5inv(x, prec, dag=dag) for x in halves])):
                check(op.unpack(*got, prec).cpu().numpy(), ref, tol, (dims, Ls, prec, dag))
    op.close()


# a hop with its directions split over wavefronts (the small lattices' default)
# against the loop variants that set_tuning asks for: fewer sites than one
# wavefront's, partial last wavefronts, odd Ls, one site per wavefront, matrix-core
# and dot-product colour multiply (Ls divisible by 4 or not)
@pytest.mark.parametrize("dims,Ls,nrhs", [((2, 2, 2, 2), 2, 1), ((4, 2, 2, 6), 5, 3), ((6, 4, 2, 4), 33, 2),
                                          ((4, 4, 4, 6), 12, 1), ((4, 4, 6, 6), 7, 2), ((8, 8, 8, 16), 8, 1)])
def test_split_hop_same_bits(torch_cuda, dims, Ls, nrhs):
    """The split form adds the eight directions in the order of the loop: every
    operator block has the same bits, and a solve the same iterates."""
    torch = torch_cuda
    mobius, op, eta = _setup(torch, dims, Ls, nrhs)
    fields = {}
    for prec in (mobius.F64, mobius.F32, mobius.F16):
        even, odd = op.pack(eta, prec, nrhs)
        fields[prec] = {p: torch.cat([even, odd]) if p == mobius.OP_FULL else odd for p in range(8)}

    def blocks():
        return {(prec, o, dag): op.dslash(fields[prec][o], 1, prec, op=o, dag=dag, nrhs=nrhs)
                for prec in fields for o in range(8) for dag in (False, True)}

    def solves():
        return [op.solve(eta, tol=1e-10, maxiter=20000, inner_prec=prec)[:2] for prec in fields]

    split, ssol = blocks(), solves() if Ls == 8 else []
    for prec in fields:
        op.set_tuning(prec, 0 if prec == mobius.F64 else 2, 1, 1, 0, mfma=1)
    loop, lsol = blocks(), solves() if Ls == 8 else []
    for key in split:
        assert torch.equal(split[key], loop[key]), key
    for (a, ia), (b, ib) in zip(ssol, lsol):
        assert torch.equal(a, b)
        assert [i.iters for i in ia] == [i.iters for i in ib]
    op.close()


def _gauss(torch, shape, seed):
    gen = torch.Generator(device="cuda").manual_seed(seed)
    return torch.view_as_complex(torch.randn(shape + (2,), dtype=torch.float64, device="cuda", generator=gen))


# right-hand sides that take turns in a workgroup on links staged once: hops without
# an I^-1 epilogue on some 400 site blocks, with one on 512 (FP32, FP16: its buffer
# lies past the links), and every hop where the links outgrow the cache (FP64)
SHARED = [((12, 12, 12, 16), 8, (0, 1, 2)), ((16, 16, 16, 16), 4, (1, 2)), ((16, 16, 16, 64), 5, (0,))]


@pytest.mark.parametrize("dims,Ls,precs", SHARED, ids=[f"{d}-Ls{ls}" for d, ls, _ in SHARED])
def test_right_hand_sides_sharing_links_same_bits(torch_cuda, dims, Ls, precs):
    """Each right-hand side has the bits of its own application, in every operator
    block; cut by maxiter, each solve form the iterates of its solo solve."""
    torch = torch_cuda
    from paper_1206_5214_amd import inputs, mobius
    n = 2
    U = torch.from_numpy(inputs.random_links(dims, 0.4, np.random.default_rng(3))).cuda()
    op = mobius.Operator(dims, Ls, 1.8, 0.05, 1.5, 0.5, U)
    eta = _gauss(torch, op.canon_shape(n), 4)
    if dims == (16, 16, 16, 64):  # the others: their hop mixes its input or has no epilogue
        assert op.hop_flags(precs[0], n) & mobius.HOP_SHARED_LINKS
    for prec in precs:
        full = op.pack_full(eta, prec, n)
        one = [op.pack_full(eta[r], prec) for r in range(n)]
        fb = op.field_bytes(prec)
        for o in range(8):
            for dag in (False, True):
                got = op.dslash(full if o == mobius.OP_FULL else full[n * fb:], 1, prec, op=o, dag=dag, nrhs=n)
                for r in range(n):
                    want = op.dslash(one[r] if o == mobius.OP_FULL else one[r][fb:], 1, prec, op=o, dag=dag)
                    halves = (r, n + r) if o == mobius.OP_FULL else (r,)
                    for k, h in enumerate(halves):
                        assert torch.equal(got[h * fb:(h + 1) * fb], want[k * fb:(k + 1) * fb]), (prec, o, dag, r)
        del full, one, got, want
        for kw in [{"form": f} for f in range(4)] + [{"dagger": True}]:
            opts = dict(tol=1e-12, maxiter=9, inner_prec=prec, check_every=4, **kw)
            sol = op.solve(eta, **opts)[0]
            for r in range(n):
                assert torch.equal(sol[r], op.solve(eta[r], **opts)[0]), (prec, kw, r)
    op.close()


@pytest.mark.parametrize("prec", [0, 1, 2], ids=["f64", "f32", "f16"])
def test_batch_with_shared_links_same_iterates(torch_cuda, prec):
    """A batched launch in which one lattice's right-hand sides share their links (the
    I^-1 buffer then lies past the links for every lattice) and another's do not.
    FP16: the rows of a site block at Ls = 4 are too large to stage, so that the
    batch runs the dot-product loop everywhere, and the solo solves are told to."""
    torch = torch_cuda
    from paper_1206_5214_amd import inputs, mobius
    rng = np.random.default_rng(6)
    ops, srcs = [], []
    for k, (dims, Ls) in enumerate((((12, 12, 12, 16), 8), ((16, 16, 16, 16), 4), ((4, 4, 4, 6), 8))):
        U = torch.from_numpy(inputs.random_links(dims, 0.4, rng)).cuda()
        ops.append(mobius.Operator(dims, Ls, 1.8, 0.05, 1.5, 0.5, U))
        srcs.append(_gauss(torch, ops[-1].canon_shape(2), 10 + k))
    opts = dict(tol=1e-12, maxiter=9, inner_prec=prec, check_every=4)
    sols = mobius.batch_solve(ops, srcs, **opts)[0]
    for op, src, sol in zip(ops, srcs, sols):
        if prec == mobius.F16:
            op.set_tuning(prec, 2, 1, 1, 0, mfma=0)
        for r in range(2):
            assert torch.equal(sol[r], op.solve(src[r].contiguous(), **opts)[0]), (op.dims, r)
        op.close()


def _slices(Ls):
    rng = np.random.default_rng(8)
    return {"b5s": tuple(rng.uniform(1.0, 2.0, Ls)), "c5s": tuple(rng.uniform(0.0, 0.8, Ls))}


# the split form, which the small lattices of the oracle tests run by default, against
# the loop that larger ones run: constant and per-slice coefficients, a chemical
# potential (the adjoint's own links), matrix-core and dot-product FP16 loops
@pytest.mark.parametrize("dims,Ls,kw", [((4, 2, 2, 6), 8, {}), ((4, 2, 2, 6), 8, _slices(8)),
                                        ((4, 4, 2, 2), 5, _slices(5)), ((4, 2, 2, 6), 8, {"mu": 0.3}),
                                        ((4, 2, 4, 2), 5, {"mu": -0.4})],
                         ids=["const-Ls8", "slices-Ls8", "slices-Ls5", "mu-Ls8", "mu-Ls5"])
@pytest.mark.parametrize("prec", [0, 1, 2], ids=["f64", "f32", "f16"])
def test_split_and_loop_agree_in_every_operator_and_form(torch_cuda, dims, Ls, kw, prec):
    """Every operator block, the solve forms cut by maxiter and the force, of one and
    two right-hand sides, bit for bit; each side is asked which form it ran."""
    torch = torch_cuda
    mobius, op, eta = _setup(torch, dims, Ls, 2, **kw)
    full = {1: op.pack_full(eta[0].contiguous(), prec), 2: op.pack_full(eta, prec, 2)}
    fb = op.field_bytes(prec)

    def attempt(f):
        try:
            return f()
        except mobius.MobiusError as e:  # (the left forms need constant coefficients)
            return str(e)

    def everything():
        out = {}
        for n in (1, 2):
            src = eta if n == 2 else eta[0].contiguous()
            for o in range(8):
                for dag in (False, True):
                    x = full[n] if o == mobius.OP_FULL else full[n][n * fb:]
                    out[n, o, dag] = attempt(lambda: op.dslash(x, 1, prec, op=o, dag=dag, nrhs=n))
            for form in range(4):
                out[n, "solve", form] = attempt(lambda: op.solve(src, tol=1e-13, maxiter=7, inner_prec=prec,
                                                                 form=form, check_every=3)[0])
            out[n, "solve", "dagger"] = attempt(lambda: op.solve(src, tol=1e-13, maxiter=7, inner_prec=prec,
                                                                 dagger=True, check_every=3)[0])
        s, gl, gp, _, _ = op.force(eta[0].contiguous(), tol=1e-13, maxiter=7, inner_prec=prec, check_every=3)
        out["force"] = torch.cat([torch.view_as_real(t).flatten() for t in (gl, gp)] + [torch.tensor([s]).cuda()])
        return out

    assert op.hop_flags(prec, 2) & mobius.HOP_SPLIT
    split = everything()
    for p in {prec, mobius.F64}:  # (a solve's residual and the force run FP64 hops)
        op.set_tuning(p, 2 if p == mobius.F16 else 0, 1, 1, 0, mfma=1)
        assert op.hop_flags(p, 1) == op.hop_flags(p, 2) == 0
    loop = everything()
    assert sum(isinstance(v, str) for v in split.values()) <= 12
    for key in split:
        if isinstance(split[key], str):
            assert split[key] == loop[key], key
        else:
            assert torch.equal(split[key], loop[key]), key
    op.close()


@pytest.mark.parametrize("prec,blocks", [(0, 160), (1, 400), (2, 160)], ids=["f64", "f32", "f16"])
def test_split_threshold(torch_cuda, prec, blocks):
    """8 site blocks: the last number of right-hand sides that splits and the first
    that does not, each right-hand side with the bits of its own application."""
    torch = torch_cuda
    n = blocks // 8
    mobius, op, eta = _setup(torch, (4, 4, 4, 8), 8, n + 1)
    assert op.hop_flags(prec, n) & mobius.HOP_SPLIT and not op.hop_flags(prec, n + 1) & mobius.HOP_SPLIT
    fb = op.field_bytes(prec)
    _, x = op.pack(eta, prec, n + 1)
    for o in (mobius.OP_HOP, mobius.OP_SCHUR):
        one = [op.dslash(x[r * fb:(r + 1) * fb], 0 if o == mobius.OP_HOP else 1, prec, op=o) for r in range(n + 1)]
        for m in (n, n + 1):
            got = op.dslash(x, 0 if o == mobius.OP_HOP else 1, prec, op=o, nrhs=m)
            assert torch.equal(got, torch.cat(one[:m])), (o, m)
    op.close()
