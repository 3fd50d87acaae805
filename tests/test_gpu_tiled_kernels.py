"""The kernels that smaller product sets no longer reach by default: the tiled contractions with the
update in their epilogue (sets of more ordinates than the sparse step holds) and the separate Heun
stencils in FP32 (asked for), over several steps, chunk and strip edges, each asserted to be what
runs.  Bounds as for the same kernels at the sets that used to reach them."""
import numpy as np
import pytest

import workloads as wl
from gpu_util import fp32_budget_floor, gpu_run, oracle_run, rel_l2
from test_gpu_banded_lowprec import _emulated

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("needs a GPU", allow_module_level=True)
from paper_1911_08801_amd import asn  # noqa: E402


def _spec(nx, ny, n_polar, n_azim, ico=0):
    spec = wl.random_problem(nx + 3 * ny, nx, ny, n_polar=n_polar, n_azim=n_azim, beta=4.5)
    spec.ico_order = ico
    return spec, wl.random_state(nx * 7 + ny, spec.q, ny, nx)


def _runs(spec, kernel, **kw):
    p = asn.from_spec(spec, set_initial_state=False, **kw)
    assert asn.asn_step_kernel(p) == kernel
    p.close()


@pytest.mark.parametrize("nx,ny", [(61, 17), (130, 67), (1362, 3), (1363, 3), (2049, 2)])
@pytest.mark.parametrize("norm", ["sym", "row"])
def test_separate_heun_stencils_match_oracle(nx, ny, norm):
    # grids up to 1362 columns run over flat 2048-cell chunks (the second crosses several chunk
    # edges mid-row), wider ones over column strips
    spec, psi0 = _spec(nx, ny, 2, 4)
    _runs(spec, "gemm_f32_kernel<false>", scheme="heun", unfused=True, norm=norm)
    state, phi, bud, _ = gpu_run(asn, spec, 2, psi0=psi0, scheme="heun", unfused=True, norm=norm)
    ref, phi_ref, st = oracle_run(spec, 2, psi0=psi0, scheme="heun", norm=norm)
    assert np.max(np.abs(state - ref)) <= 8e-6 * np.abs(ref).max()
    assert np.max(np.abs(phi - phi_ref)) <= 8e-6 * np.abs(phi_ref).max()
    assert bud["steps"] == 2
    assert bud["max_residual"] <= max(1e-10, 64 * fp32_budget_floor(state, st.w))


@pytest.mark.parametrize("nx,ny", [(1, 1), (130, 33), (65, 17), (300, 3)])
@pytest.mark.parametrize("n_polar,n_azim,ico", [(4, 160, 0), (1, 4, 10)])
def test_fused_contraction_matches_oracle_and_separate_kernels(nx, ny, n_polar, n_azim, ico):
    spec, psi0 = _spec(nx, ny, n_polar, n_azim, ico)
    _runs(spec, "gemm_f32_kernel<true>", form="fused")
    state, phi, bud, _ = gpu_run(asn, spec, 3, psi0=psi0, form="fused")
    ref, phi_ref, st = oracle_run(spec, 3, psi0=psi0)
    assert np.max(np.abs(state - ref)) <= 8e-6 * np.abs(ref).max()
    assert np.max(np.abs(phi - phi_ref)) <= 8e-6 * np.abs(phi_ref).max()
    assert bud["max_residual"] <= max(1e-10, 64 * fp32_budget_floor(state, st.w))
    sep, phi_s, _, _ = gpu_run(asn, spec, 3, psi0=psi0, form="separate")
    assert rel_l2(state, sep) <= 1e-6 and rel_l2(phi, phi_s) <= 1e-6


@pytest.mark.parametrize("nx,ny", [(70, 33), (129, 9)])
@pytest.mark.parametrize("n_polar,n_azim,ico", [(4, 160, 0), (1, 4, 10)])
@pytest.mark.parametrize("dtype,block", [("bf16", 256), ("f16", 256), ("bf16", 64)])
def test_pending_correction_of_later_steps_matches_emulation(nx, ny, n_polar, n_azim, ico, dtype, block):
    # from the second step on the stored state lacks its pending per-cell correction
    spec, psi0 = _spec(nx, ny, n_polar, n_azim, ico)
    _runs(spec, "gemm_lp_kernel<%d, true>" % {"bf16": 1, "f16": 2}[dtype], form="fused", dtype=dtype)
    one, _, _, _ = gpu_run(asn, spec, 1, psi0=psi0, dtype=dtype, form="fused", scale_block=block)
    ref, _ = _emulated(spec, 1, psi0, dtype, block)
    assert np.max(np.abs(one - ref)) <= 2e-6 * np.abs(ref).max()
    state, phi, bud, _ = gpu_run(asn, spec, 4, psi0=psi0, dtype=dtype, form="fused", scale_block=block)
    ref, st = _emulated(spec, 4, psi0, dtype, block)
    assert rel_l2(state, ref) <= 1e-5
    assert bud["steps"] == 4
    assert bud["max_residual"] <= max(1e-10, 64 * fp32_budget_floor(state, st.w))


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_fused_batches_equal_alone_bitwise(dtype):
    specs = [_spec(nx, ny, 4, 160)[0] for nx, ny in ((40, 30), (17, 5), (64, 64))]
    alone = []
    for s in specs:
        p = asn.from_spec(s, dtype=dtype, form="fused")
        asn.asn_step(p, 5)
        alone.append((asn.asn_get_state(p), asn.asn_scalar_flux(p), asn.asn_mass_budget(p)))
        p.close()
    for step in (asn.asn_step_batch, asn.asn_step_batch_noalloc):
        probs = [asn.from_spec(s, dtype=dtype, form="fused") for s in specs]
        step(probs, 2)
        step(probs, 3)
        for p, (state, phi, bud) in zip(probs, alone):
            assert np.array_equal(asn.asn_get_state(p), state)
            assert np.array_equal(asn.asn_scalar_flux(p), phi)
            assert asn.asn_mass_budget(p) == bud
            p.close()
