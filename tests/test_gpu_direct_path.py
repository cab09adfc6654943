"""The direct contraction's kernels, at the sizes for which the fast
evaluation is chosen otherwise: what the library runs above 2048^2, where the
grids do not fit, and wherever a few visibilities make it the faster path.
The checks are those of the files that test either path; here UVMEM_DFT, read
at finalize, asks for the contraction, and every context must have it."""
import numpy as np
import pytest
import torch

import test_gpu_fullsize as full
import test_gpu_imaging as imaging
import test_gpu_parity as parity
import test_gpu_shared as shared
from _common import TOL, Problem, flush, rel
from paper_1703_02920_amd import uvmem

pytestmark = pytest.mark.gpu
PRECS = ["fp64", "fp32", "bf16x3", "fp16x3"]


@pytest.fixture
def direct(monkeypatch):
    """The contraction for every context made in the test; the contexts'
    info() after the test."""
    infos = []
    finalize = uvmem.Context.finalize

    def recorded(self):
        finalize(self)
        infos.append(self.info())
        return self

    monkeypatch.setenv("UVMEM_DFT", "direct")
    monkeypatch.setattr(uvmem.Context, "finalize", recorded)
    yield infos
    assert infos and all(i["transform_side"] == 0 for i in infos)


@pytest.mark.parametrize("prec", PRECS)
@pytest.mark.parametrize("n,nvis", [(128, 777), (100, 321), (256, 1203)])
def test_forward_and_adjoint(direct, prec, n, nvis):
    parity.test_forward_parity(prec, n, nvis)
    parity.test_adjoint_parity(prec, n, nvis)


@pytest.mark.parametrize("prec", ["fp32", "bf16x3", "fp16x3"])
def test_short_last_round(direct, prec):
    parity.test_forward_parity_short_last_round(prec)


@pytest.mark.parametrize("prec", PRECS)
def test_every_visibility_and_pixel_256(direct, prec):
    """256^2 x 99,840: split-K chunks of the FP32 and split adjoints."""
    full.test_c2_full_phi_grad(prec)


@pytest.mark.parametrize("prec", PRECS)
def test_long_chunks_512(direct, prec):
    full.test_c3_sampled_and_point_source(prec)


@pytest.mark.parametrize("prec", PRECS)
def test_uneven_channels_256(direct, prec):
    full.test_c4_batched_sampled_and_point_source(prec)


@pytest.mark.parametrize("prec", ["fp32", "bf16x3", "fp16x3"])
def test_long_chunks_1024(direct, prec):
    """1024^2 x 5,000,250: FP32 sums folded within a chunk, the longest
    chunks of the split adjoint."""
    full.test_c5_sampled_and_point_source(prec)


@pytest.mark.parametrize("prec", ["fp32", "fp16x3"])
def test_shared_image(direct, prec):
    full.test_c4_shared_sampled_and_point_source(prec)
    shared.test_shared_phi_grad_parity(prec, "ragged")


@pytest.mark.parametrize("prec", PRECS)
def test_dirty_image(direct, prec):
    imaging.test_dirty_image_and_psf_parity(prec, "cube")


@pytest.mark.parametrize("prec", ["fp64", "fp32", "bf16x3"])
def test_focus_region(direct, prec):
    imaging.test_focus_region_visits_fewer_tiles(prec)
    assert 0 < direct[0]["n_fwd_wgs_region"] <= direct[0]["n_fwd_wgs"]


@pytest.mark.parametrize("prec,n", [("fp64", 256), ("fp32", 512), ("bf16x3", 512), ("fp16x3", 512)])
def test_focus_region_of_one_adjoint_tile(direct, prec, n):
    """A region inside one of four adjoint tiles: three are left out, the
    gradient inside is the oracle's, outside it is zero."""
    prob = Problem.random(n, [600], seed=67)
    ch = prob.chans[0]
    free = np.zeros((n, n), bool)
    free[n // 2 + 5:n // 2 + 90, 17:101] = True
    ctx = uvmem.Context(n, 1, prec)
    ctx.set_uv(0, ch["u"], ch["v"], prob.cell)
    ctx.set_vis(0, ch["vis"])
    ctx.set_weights(0, ch["w"])
    ctx.set_beam(0, ch["fwhm"])
    ctx.set_mask(0, free)
    ctx.set_prior(prob.M, prob.lam)
    ctx.finalize()
    info = direct[-1]
    tile = info["adj_tile"]
    assert n == 2 * tile and 4 * info["n_adj_wgs_region"] <= 2 * info["n_adj_items"]
    I = torch.tensor(np.random.default_rng(4).uniform(1e-3, 1.0, (1, n, n)), dtype=ctx.dtype, device="cuda")
    scal, grad = ctx.phi_and_grad(I)
    r = prob.oracle_phi_grad(0, I.cpu().numpy()[0].astype(np.float64))
    g = grad.cpu().numpy()[0]
    e_g, e_p = rel(g[free], r["grad"][free]), abs(float(scal[0, 0]) - r["phi"]) / abs(r["phi"])
    J = ctx.image()
    ctx.cg_init(J, init_to_floor=True)
    ctx.cg_run(J, 2, graph=False)
    Jn = J.cpu().numpy()[0]
    flush(f"region of one tile {prec} {n}^2: grad {e_g:.2e} phi {e_p:.2e}, "
          f"{info['n_adj_wgs_region']} of {info['n_adj_items']} adjoint workgroups")
    assert max(e_g, e_p) < TOL[prec] and np.all(g[~free] == 0.0)
    assert np.all(Jn[~free] == Jn[0, 0]) and Jn[free].max() > Jn[0, 0]
