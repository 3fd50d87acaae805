"""GPU parity of the step that keeps every ordinate of 64 cells in LDS and multiplies the
nonzeros of any K (icosahedron sets, product sets without a banded kernel), against the
oracle on the same seeded inputs, and of what lies beyond its limits (a dense K of many
ordinates, more ordinates than LDS holds)."""
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

# (n_polar, n_azim, icosahedron order, beta): one ordinate group and a part of one, groups filled
# up (42, 162 ordinates), 16 waves (362), dense K of 162 and (too dense) 252 ordinates, as many
# as LDS holds (632) and more (640, 812); product sets
SETS = [(1, 2, 0, 4.5), (3, 2, 0, 4.5), (1, 4, 2, 4.5), (1, 4, 3, 4.5), (1, 4, 5, 4.5), (1, 4, 7, 4.5),
        (1, 4, 5, 80.0), (1, 4, 6, 80.0), (1, 4, 10, 4.5), (5, 10, 0, 4.5), (8, 16, 0, 6.0), (4, 158, 0, 4.5), (4, 160, 0, 4.5)]
GRIDS = [(1, 1), (3, 70), (63, 2), (64, 3), (65, 4)]


def _spec(nx, ny, n_polar, n_azim, ico, beta):
    spec = wl.random_problem(nx + ny + n_azim + ico, nx, ny, n_polar=n_polar, n_azim=n_azim, beta=beta)
    spec.ico_order = ico
    return spec, wl.random_state(nx + n_polar, spec.q, ny, nx)


@pytest.mark.parametrize("nx,ny", GRIDS)
@pytest.mark.parametrize("n_polar,n_azim,ico,beta", SETS)
@pytest.mark.parametrize("scheme", ["euler", "heun"])
def test_two_steps_match_oracle(nx, ny, n_polar, n_azim, ico, beta, scheme):
    spec, psi0 = _spec(nx, ny, n_polar, n_azim, ico, beta)
    state, phi, bud, _ = gpu_run(asn, spec, 2, psi0=psi0, scheme=scheme)
    ref, phi_ref, st = oracle_run(spec, 2, psi0=psi0, scheme=scheme)
    assert np.max(np.abs(state - ref)) <= 8e-6 * np.abs(ref).max()
    assert np.max(np.abs(phi - phi_ref)) <= 8e-6 * np.abs(phi_ref).max()
    assert bud["steps"] == 2
    assert bud["max_residual"] <= max(1e-10, 64 * fp32_budget_floor(state, st.w))


@pytest.mark.parametrize("nx,ny,block", [(1, 1, 256), (63, 2, 64), (65, 4, 256), (130, 40, 4096)])
@pytest.mark.parametrize("n_polar,n_azim,ico,beta", [(1, 2, 0, 4.5), (1, 4, 3, 4.5), (1, 4, 7, 4.5), (1, 4, 6, 80.0),
                                                     (8, 16, 0, 4.5), (4, 158, 0, 4.5), (4, 160, 0, 4.5)])
@pytest.mark.parametrize("dtype", ["bf16", "f16"])
def test_reduced_precision_step_matches_emulation(nx, ny, block, n_polar, n_azim, ico, beta, dtype):
    spec, psi0 = _spec(nx, ny, n_polar, n_azim, ico, beta)
    state, _, _, _ = gpu_run(asn, spec, 1, psi0=psi0, dtype=dtype, scale_block=block)
    ref, _ = _emulated(spec, 1, psi0, dtype, block)
    assert np.max(np.abs(state - ref)) <= 2e-6 * np.abs(ref).max()


@pytest.mark.parametrize("scheme,dtype", [("euler", "f32"), ("euler", "bf16"), ("heun", "f32")])
def test_batch_of_all_kinds_equals_alone_bitwise(scheme, dtype):
    # 8 and 16 waves, beyond the limits, and (Heun) a banded one, in an order that interleaves them
    sets = [(1, 4, 10, 4.5), (1, 4, 5, 4.5), (1, 4, 7, 4.5), (1, 4, 6, 80.0), (5, 10, 0, 4.5), (4, 8, 0, 4.5)]
    specs = [_spec(20 + 13 * i, 9 + i, *s)[0] for i, s in enumerate(sets)]
    kw = dict(dtype=dtype, scheme=scheme, form="fused")
    limits = [5, 2, 7, 4, 3, 6]
    alone = []
    for spec, n in zip(specs, limits):
        p = asn.from_spec(spec, **kw)
        asn.asn_step(p, n)
        alone.append((asn.asn_get_state(p), asn.asn_scalar_flux(p), asn.asn_mass_budget(p)))
        p.close()
    with torch.cuda.stream(torch.cuda.Stream()):
        probs = [asn.from_spec(s, **kw) for s in specs]
        b = asn.asn_batch_create(probs)
        for k in range(2):
            asn.asn_batch_step(b, 4, limits=[max(0, n - 4 * k) for n in limits])
        for p, (state, phi, bud), n in zip(probs, alone, limits):
            assert asn.asn_info(p)["steps_done"] == n
            assert np.array_equal(asn.asn_get_state(p), state)
            assert np.array_equal(asn.asn_scalar_flux(p), phi)
            assert asn.asn_mass_budget(p) == bud
        b.close()
        for p in probs:
            p.close()
    torch.cuda.synchronize()


def test_automatic_form_equals_separate_kernels():
    # 350^2 x 362 cell-ordinates: reported as separate kernels
    spec, _ = _spec(350, 350, 1, 4, 7, 4.5)
    state, phi, _, _ = gpu_run(asn, spec, 2, form="auto")
    sep, phi_s, _, _ = gpu_run(asn, spec, 2, form="separate")
    assert rel_l2(state, sep) <= 1e-6 and rel_l2(phi, phi_s) <= 1e-6


@pytest.mark.parametrize("large,small,dtype", [((4, 158, 0, 4.5), (1, 4, 7, 4.5), "f32"),
                                               ((4, 158, 0, 4.5), (1, 4, 7, 4.5), "bf16"),
                                               ((1, 4, 6, 4.5), (1, 4, 2, 4.5), "f32"),
                                               ((2, 64, 0, 4.5), (2, 32, 0, 4.5), "f16")])
def test_larger_problem_steps_after_a_smaller_one_is_created(large, small, dtype):
    # one kernel instance serves both (sparse of 16 waves: 158 and 91 KiB of LDS, of 8 waves: 63 and
    # 10; banded: 66 and 33), whose limit for LDS a problem's creation must not lower
    spec, psi0 = _spec(65, 4, *large)
    state, _, _, _ = gpu_run(asn, spec, 2, psi0=psi0, dtype=dtype, form="auto")
    p = asn.from_spec(spec, dtype=dtype, set_initial_state=False)
    asn.asn_set_state(p, psi0)
    q = asn.from_spec(_spec(9, 5, *small)[0], dtype=dtype)
    asn.asn_step(q, 1)
    asn.asn_step(p, 2)
    assert np.array_equal(asn.asn_get_state(p), state)
    p.close()
    q.close()


@pytest.mark.parametrize("n,n_polar,n_azim,ico,beta,dtype,scheme,kernel", [
    (200, 2, 64, 0, 80.0, "bf16", "euler", "sparse"), (500, 2, 64, 0, 80.0, "bf16", "euler", "gemm_lp_kernel<1, true>"),
    (500, 2, 64, 0, 80.0, "f32", "euler", "gemm_f32_kernel<true>"), (500, 2, 64, 0, 4.5, "bf16", "euler", "sparse"),
    (200, 1, 4, 5, 80.0, "f16", "euler", "sparse"), (500, 1, 4, 5, 80.0, "f16", "euler", "gemm_lp_kernel<2, true>"),
    (500, 1, 4, 5, 80.0, "f32", "euler", "sparse"), (500, 1, 4, 5, 10.0, "bf16", "euler", "sparse"),
    (200, 16, 32, 0, 7.0, "bf16", "euler", "sparse"), (500, 16, 32, 0, 7.0, "bf16", "euler", "gemm_lp_kernel<1, true>"),
    (500, 16, 32, 0, 7.0, "f32", "euler", "sparse"), (500, 8, 64, 0, 13.0, "f16", "euler", "gemm_lp_kernel<2, true>"),
    (500, 1, 4, 8, 7.0, "bf16", "euler", "sparse"), (400, 4, 32, 0, 40.0, "f32", "heun", "gemm_f32_kernel<false>"),
    (800, 4, 32, 0, 40.0, "f32", "heun", "sparse")])
def test_the_faster_kernel_is_taken(n, n_polar, n_azim, ico, beta, dtype, scheme, kernel):
    # both measured, 3 to 30 % apart: large problems with a K that is dense for their ordinates
    # go to the tiled contraction
    spec = wl.random_problem(3, n, n, n_polar=n_polar, n_azim=n_azim, beta=beta)
    spec.ico_order = ico
    p = asn.from_spec(spec, dtype=dtype, scheme=scheme, form="fused", set_initial_state=False)
    assert asn.asn_step_kernel(p).startswith(kernel)
    p.close()


def test_batch_of_sizes_that_take_different_kernels_equals_alone_bitwise():
    specs = [_spec(nx, ny, 2, 64, 0, 80.0)[0] for nx, ny in ((20, 9), (330, 330), (64, 3))]
    kw = dict(dtype="bf16", form="fused")
    alone = []
    for spec in specs:
        p = asn.from_spec(spec, **kw)
        asn.asn_step(p, 3)
        alone.append((asn.asn_get_state(p), asn.asn_mass_budget(p)))
        p.close()
    probs = [asn.from_spec(s, **kw) for s in specs]
    assert [asn.asn_step_kernel(p)[:6] for p in probs] == ["sparse", "gemm_l", "sparse"]
    asn.asn_step_batch(probs, 3)
    for p, (state, bud) in zip(probs, alone):
        assert np.array_equal(asn.asn_get_state(p), state)
        assert asn.asn_mass_budget(p) == bud
        p.close()
