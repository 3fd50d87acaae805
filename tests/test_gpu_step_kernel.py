"""The kernel that asn_step_kernel names is the one that a form, set and grid lead to."""
import pytest

import workloads as wl

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("needs a GPU", allow_module_level=True)
from paper_1911_08801_amd import asn  # noqa: E402


def kernel_of(nx, ny, n_polar, n_azim, ico=0, beta=4.5, **kw):
    spec = wl.random_problem(3, nx, ny, n_polar=n_polar, n_azim=n_azim, beta=beta)
    spec.ico_order = ico
    p = asn.from_spec(spec, set_initial_state=False, **kw)
    name, form = asn.asn_step_kernel(p), asn.asn_step_form(p)
    p.close()
    return name, form


@pytest.mark.parametrize("args,kw,expected", [
    ((37, 21, 4, 8), dict(form="auto"), ("banded_euler_kernel<2, 1024, 0, 0>", "banded")),
    ((37, 21, 4, 8), dict(form="fused"), ("sparse_step_kernel<0, 0, 512>", "fused")),
    ((37, 21, 4, 8), dict(form="separate"), ("gemm_f32_kernel<false>", "separate")),
    ((37, 21, 4, 8), dict(form="auto", scheme="heun"), ("banded_euler_kernel<2, 1024, 0, 1>", "separate")),
    ((37, 21, 4, 8), dict(form="separate", scheme="heun"), ("gemm_f32_kernel<false>", "separate")),
    ((37, 21, 1, 4, 5), dict(form="auto", scheme="heun"), ("sparse_step_kernel<0, 1, 512>", "separate")),
    ((37, 21, 16, 32), dict(form="auto", dtype="bf16"), ("banded_euler_kernel<2, 1024, 1, 0>", "banded")),
    ((37, 21, 4, 158), dict(form="fused", dtype="f16"), ("sparse_step_kernel<2, 0, 1024>", "fused")),
    ((37, 21, 4, 160), dict(form="fused", dtype="f16"), ("gemm_lp_kernel<2, true>", "fused")),
    ((37, 21, 4, 160), dict(form="fused"), ("gemm_f32_kernel<true>", "fused")),
    ((37, 21, 1, 4, 2), dict(scheme="implicit"), ("", "separate")),
])
def test_kernel_of_a_problem(args, kw, expected):
    assert kernel_of(*args, **kw) == expected
