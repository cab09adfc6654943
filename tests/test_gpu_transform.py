"""The fast evaluation of the direct DFT (oversampled transform) against the
oracle and against the direct contraction.

UVMEM_DFT=transform / direct, read at finalize, forces either path.  Bars:
the fast evaluation is held to the same tolerances as the direct kernels
(FP64: rounding of FP64 sums, 1e-12; below FP64: the FP32 bar 1e-6 in every
precision.  In FP32 it has to cover the window error, about 1e-8, and FP32
adjoint tiles and half spectra around FP64 sums; in the split precisions FP32
windows, tile products, the sums of up to 1,024 visibilities of an item, grids
and tiles, whose rounding the window's correction magnifies up to eleven times
in the corners of the image).
"""
import os

import numpy as np
import pytest
import torch

from _common import TOL, Problem, flush, rel
from paper_1703_02920_amd import synth

pytestmark = pytest.mark.gpu
BAR = {"fp64": TOL["fp64"], "fp32": TOL["fp32"], "bf16x3": TOL["fp32"], "fp16x3": TOL["fp32"]}


def _context(prob, prec, path, mode="cube", masks=None):
    assert torch.cuda.is_available(), "needs a GPU"
    from paper_1703_02920_amd.uvmem import Context
    old = os.environ.get("UVMEM_DFT")
    os.environ["UVMEM_DFT"] = path
    try:
        ctx = Context(prob.n, prob.n_chan, prec, mode=mode)
        for c, ch in enumerate(prob.chans):
            ctx.set_uv(c, ch["u"], ch["v"], prob.cell)
            ctx.set_vis(c, ch["vis"])
            ctx.set_weights(c, ch["w"])
            ctx.set_beam(c, ch["fwhm"])
            if ch.get("x0", 0.0) or ch.get("y0", 0.0):
                ctx.set_phase_centre(c, ch["x0"], ch["y0"])
        if masks is not None:
            ctx.set_mask(0, masks)
        ctx.set_prior(prob.M, prob.lam)
        ctx.finalize()
    finally:
        if old is None:
            del os.environ["UVMEM_DFT"]
        else:
            os.environ["UVMEM_DFT"] = old
    assert (ctx.info()["transform_side"] > 0) == (path == "transform")
    return ctx


def _edges(prob, side):
    """Coordinates at the edges of the fast evaluation's bookkeeping: zero,
    half a cycle, exact nodes, midway between nodes, the last bin column,
    negative a, and whole cycles beyond the first."""
    ch = prob.chans[0]
    e = [0.0, 0.5, -0.5, 8.0 / side, 7.5 / side, 8.5 / side, (side / 2 - 0.25) / side, -3.0 / side, 0.5 - 1e-12,
         3.25, -2.75, 1.0, -1e-300, 16.0 / side, 15.5 / side]
    pairs = [(x, y) for x in e for y in e][: len(ch["u"])]
    ch["u"][: len(pairs)] = np.array([p[0] for p in pairs]) / prob.cell
    ch["v"][: len(pairs)] = np.array([p[1] for p in pairs]) / prob.cell


@pytest.mark.parametrize("prec", ["fp64", "fp32", "bf16x3", "fp16x3"])
@pytest.mark.parametrize("n,nvis", [(2, [1]), (32, [300]), (34, [65, 0, 33]), (64, [700]), (100, [333]),
                                    (256, [500]), (514, [260]), (1026, [230])])
def test_transform_matches_oracle(prec, n, nvis):
    """Every transform length (64 .. 4096), ragged sides, single and empty
    channels, and coordinates at the edges of bins and of the half plane."""
    flush(f"transform vs oracle {prec} n={n} nvis={nvis}")
    prob = Problem.random(n, nvis, seed=500 + n)
    side = max(64, 1 << (2 * n - 1).bit_length())
    _edges(prob, side)
    ctx = _context(prob, prec, "transform")
    assert ctx.info()["transform_side"] == side
    img = np.stack([np.random.default_rng(7 + c).uniform(1e-3, 1.0, (n, n)) for c in range(len(nvis))])
    I = torch.tensor(img, dtype=ctx.dtype, device="cuda")
    img = I.cpu().numpy().astype(np.float64)
    V = ctx.forward(I).cpu().numpy()
    ref = np.concatenate([prob.oracle_forward(c, img[c]) for c in range(len(nvis))])
    rng = np.random.default_rng(3)
    coef = rng.normal(size=ctx.ztot) + 1j * rng.normal(size=ctx.ztot)
    adj = ctx.adjoint(torch.tensor(coef, device="cuda")).cpu().numpy()
    scal, grad = ctx.phi_and_grad(I)
    R = ctx.residual().cpu().numpy()
    vis = np.concatenate([ch["vis"] for ch in prob.chans])
    e_v, e_r = rel(V, ref), rel(R, ref - vis)
    o = prob.offsets()
    for c in range(len(nvis)):
        e_a = rel(adj[c], prob.oracle_adjoint(c, coef[o[c]:o[c + 1]])) if nvis[c] else float(np.abs(adj[c]).max())
        r = prob.oracle_phi_grad(c, img[c])
        e_g = rel(grad.cpu().numpy()[c], r["grad"])
        e_p = abs(float(scal[c, 0]) - r["phi"]) / abs(r["phi"])
        flush(f"  channel {c}: V {e_v:.2e} R {e_r:.2e} adjoint {e_a:.2e} grad {e_g:.2e} phi {e_p:.2e}")
        assert max(e_v, e_r, e_a, e_g, e_p) < BAR[prec]
    ctx.check()


@pytest.mark.parametrize("prec", ["fp64", "fp32"])
def test_transform_dense_and_sparse_bins(prec):
    """Thousands of visibilities on one spot (several items of one bin, summed
    in order), isolated ones elsewhere; two evaluations agree bit for bit."""
    n = 64
    prob = Problem.random(n, [3001], seed=77)
    ch = prob.chans[0]
    rng = np.random.default_rng(5)
    ch["u"][:2900] = (0.1 + 1e-4 * rng.uniform(-1, 1, 2900)) / prob.cell
    ch["v"][:2900] = (-0.2 + 1e-4 * rng.uniform(-1, 1, 2900)) / prob.cell
    flush(f"transform dense bins {prec}")
    img = rng.uniform(1e-3, 1.0, (1, n, n))
    out = []
    for _ in range(2):
        ctx = _context(prob, prec, "transform")
        I = torch.tensor(img, dtype=ctx.dtype, device="cuda")
        s, g = ctx.phi_and_grad(I)
        out.append((s.cpu(), g.cpu()))
    assert torch.equal(out[0][0], out[1][0]) and torch.equal(out[0][1], out[1][1])
    r = prob.oracle_phi_grad(0, I.cpu().numpy()[0].astype(np.float64))
    e_g, e_p = rel(out[0][1].numpy()[0], r["grad"]), abs(float(out[0][0][0, 0]) - r["phi"]) / abs(r["phi"])
    flush(f"  grad {e_g:.2e} phi {e_p:.2e}")
    assert max(e_g, e_p) < BAR[prec]


@pytest.mark.parametrize("mode", ["cube", "shared"])
def test_transform_and_direct_agree_everywhere(mode):
    """The two paths on one FP64 problem (pointings with their own centres,
    an empty channel, a mask): forward, adjoint, residual and dirty image in
    the caller's order, CG steps replayed as a graph, and a checkpoint taken
    on one path and resumed on the other."""
    n, nvis = 72, [400, 0, 123]
    prob = Problem.random(n, nvis, seed=11)
    for c, ch in enumerate(prob.chans):
        ch["x0"], ch["y0"] = (3.0 * c - 2.0) * prob.cell, (1.0 - c) * prob.cell
    mask = np.zeros((n, n), bool)
    mask[10:60, 5:66] = True
    flush(f"transform vs direct {mode}")
    got = {}
    for path in ("transform", "direct"):
        ctx = _context(prob, "fp64", path, mode=mode, masks=mask)
        rng = np.random.default_rng(1)
        I = torch.tensor(rng.uniform(1e-3, 1.0, (ctx.n_img, n, n)), device="cuda")
        coef = torch.tensor(rng.normal(size=ctx.ztot) + 1j * rng.normal(size=ctx.ztot), device="cuda")
        s, g = ctx.phi_and_grad(I)
        R = ctx.residual()
        dirty, psf = ctx.dirty_image()
        J = ctx.image()
        ctx.cg_init(J, init_to_floor=True)
        hist = ctx.cg_run(J, 3, graph=True).clone()
        blob = ctx.get_state()
        got[path] = dict(ctx=ctx, blob=blob, J=J.clone(), out=[s[:, :3], g, R, dirty, psf, ctx.forward(I),
                                                               ctx.adjoint(coef), J, hist[:, :, 0]])
    for k, (x, y) in enumerate(zip(got["transform"]["out"], got["direct"]["out"])):
        e = rel(x.cpu().numpy(), y.cpu().numpy())
        flush(f"  output {k}: {e:.2e}")
        assert e < 1e-10 if k >= 7 else e < TOL["fp64"]
    ends = []
    for frm, to in (("transform", "direct"), ("direct", "transform"), ("direct", "direct")):
        ctx = got[to]["ctx"]
        J = got[frm]["J"].clone()
        ctx.cg_init(J, init_to_floor=False)
        ctx.set_state(got[frm]["blob"])
        ctx.cg_run(J, 2, graph=False)
        ends.append(J.cpu().numpy())
    assert rel(ends[0], ends[2]) < 1e-10 and rel(ends[1], ends[2]) < 1e-10


@pytest.mark.parametrize("prec", ["fp32", "bf16x3", "fp16x3"])
def test_direct_short_last_round(prec):
    """The direct forward's short last round of wave tiles (split across the
    waves of a workgroup), reached whatever the choice of path is."""
    n, tv = 256, 16 if prec == "fp32" else 32
    for nvis in (20001, 35961, 28001, 44001):
        prob = Problem.random(n, [nvis], seed=91)
        ctx = _context(prob, prec, "direct")
        info = ctx.info()
        nwg = info["n_fwd_wgs"] // info["n_fwd_parts"]
        ntiles = -(-nvis // tv)
        nfull = ntiles // (8 * nwg) * (8 * nwg)
        if 0 < ntiles - nfull <= 2 * nwg:
            break
    else:
        pytest.fail("no tried size leaves a short last round")
    I = torch.tensor(synth.random_image(n, 6, lo=1e-3, hi=1.0)[:1], dtype=ctx.dtype, device="cuda")
    V = ctx.forward(I).cpu().numpy()
    ref = prob.oracle_forward(0, I.cpu().numpy()[0].astype(np.float64))
    tail = slice(nfull * tv, nvis)
    assert rel(V, ref) < TOL[prec] and rel(V[tail], ref[tail]) < TOL[prec]


@pytest.mark.parametrize("path,n", [("direct", 180), ("direct", 182), ("transform", 182), ("transform", 530)])
def test_every_partial_is_counted(path, n):
    """Per-image reductions on either side of the number of workgroups from
    which they arrive on several counters (127 and 130 pixel blocks; 133 row
    blocks): the scalars of a CG step are those of its image.  Bar: the
    residuals were carried over the steps, FP64 rounding of two of them."""
    prob = Problem.random(n, [300, 200], seed=21)
    ctx = _context(prob, "fp64", path)
    J = ctx.image()
    ctx.cg_init(J, init_to_floor=True)
    hist = ctx.cg_run(J, 2, graph=False).clone()
    scal, _ = ctx.phi_and_grad(J)
    got, want = hist[-1].cpu().numpy()[:, :3], scal.cpu().numpy()[:, :3]
    flush(f"arrivals {path} n={n}: {rel(got, want):.2e}")
    assert rel(got, want) < 1e-10


@pytest.mark.parametrize("nvis", [[300], [300, 200]])
def test_phi_function_result_is_a_tensor_of_its_own(nvis):
    """One image and several: the value is the sum of Phi, may be changed in
    place by the caller, and its gradient is the evaluation's (exactly: the
    same kernels, scaled by a power of two)."""
    from paper_1703_02920_amd.uvmem import PhiFunction
    ctx = _context(Problem.random(64, nvis, seed=31), "fp32", "transform")
    I = torch.full((len(nvis), 64, 64), 0.3, dtype=ctx.dtype, device="cuda", requires_grad=True)
    scal, grad = ctx.phi_and_grad(I.detach())
    loss = PhiFunction.apply(I, ctx)
    assert not loss._is_view() and loss.shape == () and loss.item() == scal[:, 0].sum().item()
    loss *= 0.5
    loss.backward()
    assert I.grad.dtype == ctx.dtype and torch.equal(I.grad, 0.5 * grad)
