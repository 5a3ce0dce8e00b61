"""GPU parity of dg_apply_convective against the CPU oracle (through the C ABI).

FP64 within 1e-12 relative (2-norm), FP32 within 1e-5 relative against the
oracle applied to the FP32-rounded input.  Includes the Taylor-Green + noise
case (16^3, k=5), all degrees on ragged multi-batch meshes, small and
anisotropic meshes, the LLF coefficient, momentum conservation and constant
states on the GPU output, and the degree-sweep size on sampled elements.
"""
import numpy as np
import pytest
import torch

from gpu_common import announce, rel_err, round_f32, to_dev
from oracle import basis, mesh as M
from oracle.convective import convective_apply
from paper_1802_01439_amd import dgmf, inputs

pytestmark = pytest.mark.gpu


def _run(k, n_el, length, u, dtype=torch.float64, **kw):
    d = dgmf.make_desc(k, n_el, length, **kw)
    y = dgmf.apply_convective(d, to_dev(u, dtype))
    torch.cuda.synchronize()
    return y.double().cpu().numpy()


@pytest.mark.parametrize("dtype", [torch.float64, torch.float32])
def test_config2_taylor_green(dtype):
    """16^3 elements, k=5, 3/2-rule quadrature (m=8), TGV + N(0, 0.01^2) noise."""
    k, N = 5, 16
    msh = M.cube(N)
    u = inputs.tgv_plus_noise(basis.lgl_nodes(k), msh.n_el, msh.length, seed=inputs.FIELD_SEED_BASE + 1)
    if dtype == torch.float32:
        u = round_f32(u)
    announce(f"convective config2 k=5 N=16 {dtype}")
    y = _run(k, N, msh.length, u, dtype)
    ref = convective_apply(u, k, msh)
    assert rel_err(y, ref) < (1e-12 if dtype == torch.float64 else 1e-5)


def _mesh_for(k):
    return (3, 4, 5) if k <= 4 else (3, 2, 3)


@pytest.mark.parametrize("k", list(range(1, 12)))
def test_all_degrees_fp64(k):
    n_el = _mesh_for(k)
    length = (2 * np.pi, 2.5, 3.0)
    msh = M.Mesh(n_el, length)
    u = inputs.uniform((3, msh.N, (k + 1) ** 3), seed=400 + k)
    announce(f"convective fp64 k={k} n_el={n_el}")
    assert rel_err(_run(k, n_el, length, u), convective_apply(u, k, msh)) < 1e-12


@pytest.mark.parametrize("k", [1, 2, 4, 7, 11])
def test_all_degrees_fp32(k):
    n_el = _mesh_for(k)
    length = (2 * np.pi,) * 3
    msh = M.Mesh(n_el, length)
    u = round_f32(inputs.uniform((3, msh.N, (k + 1) ** 3), seed=500 + k))
    announce(f"convective fp32 k={k} n_el={n_el}")
    assert rel_err(_run(k, n_el, length, u, torch.float32), convective_apply(u, k, msh)) < 1e-5


@pytest.mark.parametrize("n_el,lf", [((1, 1, 1), 1.0), ((2, 1, 3), 0.5), ((2, 2, 2), 0.0), ((5, 3, 1), 2.0)])
def test_small_meshes_and_lf(n_el, lf):
    k = 3
    length = (1.0, 2.0, 0.5)
    msh = M.Mesh(n_el, length)
    u = inputs.uniform((3, msh.N, 64), seed=21)
    announce(f"convective small mesh n_el={n_el} lf={lf}")
    y = _run(k, n_el, length, u, lf_factor=lf)
    assert rel_err(y, convective_apply(u, k, msh, lf_factor=lf)) < 1e-12


def test_conservation_and_constants_on_gpu():
    k, N = 4, 6
    d = dgmf.make_desc(k, N)
    u = to_dev(inputs.uniform((3, N ** 3, 125), seed=22))
    announce("convective invariants")
    R = dgmf.apply_convective(d, u)
    sums = R.sum(dim=(1, 2)).abs().max().item()
    assert sums < 1e-12 * R.abs().sum().item()
    c = torch.ones_like(u) * torch.tensor([0.3, -0.7, 1.1], dtype=u.dtype, device=u.device)[:, None, None]
    Rc = dgmf.apply_convective(d, c.contiguous())
    assert Rc.abs().max().item() < 1e-13
    R2 = dgmf.apply_convective(d, u)
    assert torch.equal(R, R2)


@pytest.mark.parametrize("dtype", [torch.float64, torch.float32])
def test_full_size_sampled(dtype):
    """Degree-sweep size (k=5, 43^3 elements, 5.2e7 DoFs), sampled elements."""
    k, N = 5, 43
    msh = M.cube(N)
    u = inputs.uniform((3, msh.N, 216), seed=inputs.FIELD_SEED_BASE + 2 + 10 * k)
    if dtype == torch.float32:
        u = round_f32(u)
    announce(f"convective full size k=5 N=43 {dtype}")
    y = _run(k, N, msh.length, u, dtype)
    rng = np.random.default_rng(8)
    sample = np.unique(np.concatenate([rng.integers(0, msh.N, 150), [0, N - 1, N * N - 1, msh.N - 1]]))
    ref = convective_apply(u, k, msh, elems=sample)
    tol = 1e-12 if dtype == torch.float64 else 1e-5
    assert rel_err(y[:, sample], ref) < tol


@pytest.mark.parametrize("k,n_el", [(6, (7, 9, 13)), (9, (7, 7, 7)), (10, (5, 6, 9)), (11, (4, 7, 10)),
                                    (6, (3, 1, 3)), (9, (5, 1, 1)), (11, (3, 1, 4))])
def test_persistent_batch_walk_fp64(k, n_el):
    """FP64 k = 11 runs one persistent workgroup per CU that walks its XCD's
    share of element batches, loading the next batch while it finishes the
    current one: more batches than compute units, shares of unequal length,
    grids of fewer than 8 and of 8..16 workgroups.  FP64 k = 9, 10 (one
    workgroup per CU, one batch each) and k = 6 (two elements per batch) on
    meshes of the same kind, k = 6 with a ragged last batch (819 = 2 * 409 + 1,
    9 = 2 * 4 + 1).  Anisotropic box; sampled elements include the first and
    last of the mesh and an x row end."""
    length = (2 * np.pi, 1.5, 2.5)
    msh = M.Mesh(n_el, length)
    n3 = (k + 1) ** 3
    u = inputs.uniform((3, msh.N, n3), seed=1100 + k)
    announce(f"convective persistent fp64 k={k} n_el={n_el}")
    y = _run(k, n_el, length, u, lf_factor=0.8)
    nel = msh.N
    rng = np.random.default_rng(1200 + k)
    fixed = [0, 1, n_el[0] - 1, nel // 2, nel - 3, nel - 2, nel - 1]
    sample = np.unique(np.concatenate([fixed, rng.integers(0, nel, 40)]))
    ref = convective_apply(u, k, msh, lf_factor=0.8, elems=sample)
    ys = y[:, sample]
    assert rel_err(ys, ref) < 1e-12
    assert np.abs(ys - ref).max() <= 1e-11 * np.abs(ref).max()


@pytest.mark.parametrize("k,dtype", [(3, torch.float64), (9, torch.float64), (3, torch.float32), (7, torch.float32),
                                     (11, torch.float32)])
def test_input_alignment(k, dtype):
    """Pencils of contiguous values are read in 16-byte loads when the input
    is 16-byte aligned; an input one value off that (8 resp. 4 bytes) takes
    the plain loads and gives the same result bit for bit; both match the
    oracle."""
    n_el = (3, 2, 3)
    msh = M.Mesh(n_el, (2 * np.pi,) * 3)
    u = inputs.uniform((3, msh.N, (k + 1) ** 3), seed=1300 + k)
    if dtype == torch.float32:
        u = round_f32(u)
    d = dgmf.make_desc(k, n_el, msh.length)
    ua = to_dev(u, dtype)
    base = torch.empty(ua.numel() + 1, dtype=dtype, device=ua.device)
    um = base[1:].view(ua.shape)
    um.copy_(ua)
    assert ua.data_ptr() % 16 == 0 and um.data_ptr() % 16 != 0
    announce(f"convective alignment k={k} {dtype}")
    ya = dgmf.apply_convective(d, ua)
    ym = dgmf.apply_convective(d, um)
    assert torch.equal(ya, ym)
    tol = 1e-12 if dtype == torch.float64 else 1e-5
    assert rel_err(ya.double().cpu().numpy(), convective_apply(u, k, msh)) < tol


@pytest.mark.parametrize("n_el", [(1, 1, 1), (2, 1, 3), (1, 4, 2)])
@pytest.mark.parametrize("dtype", [torch.float64, torch.float32])
@pytest.mark.parametrize("k", list(range(4, 12)))
def test_one_component_per_thread_kernel(k, dtype, n_el):
    """k >= 4 runs one thread per pencil and component: every degree and type
    on meshes where an element is its own neighbour (1 per direction), sees
    the same neighbour on both sides (2), or has distinct ones (3, 4).
    Tolerances of this file: FP64 1e-12, FP32 1e-5."""
    length = (1.0, 2.0, 0.5)
    msh = M.Mesh(n_el, length)
    u = inputs.uniform((3, msh.N, (k + 1) ** 3), seed=1400 + k)
    if dtype == torch.float32:
        u = round_f32(u)
    announce(f"convective split k={k} {dtype} n_el={n_el}")
    y = dgmf.apply_convective(dgmf.make_desc(k, n_el, length, lf_factor=0.5), to_dev(u, dtype))
    ref = convective_apply(u, k, msh, lf_factor=0.5)
    assert rel_err(y.double().cpu().numpy(), ref) < (1e-12 if dtype == torch.float64 else 1e-5)


def test_unsupported_nq():
    d = dgmf.make_desc(3, 4, n_q=4)
    u = torch.zeros((3, 64, 64), dtype=torch.float64, device="cuda")
    with pytest.raises(dgmf.DgError) as ei:
        dgmf.apply_convective(d, u)
    assert ei.value.code == dgmf.DG_ERR_UNSUPPORTED
