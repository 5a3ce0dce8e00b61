"""The C entry points look a thread's last few operator plans up by the content
of the descriptor: a call must give the same values whatever was called before
it.  Every expected result comes from a thread of its own, which has no plan
yet; the kernels are deterministic, so the values are the same bits."""
import threading

import pytest
import torch

from paper_1802_01439_amd import dgmf

pytestmark = pytest.mark.gpu

BASE = dict(degree=2, n_el=(3, 2, 2), length=(1.0, 0.7, 1.3), n_comp=3)
# one field changed at a time, more of them than a thread keeps
CHANGES = [{}, {"n_el": (2, 3, 2)}, {"length": (0.7, 1.0, 1.3)}, {"penalty_factor": 2.0}, {"scale": 0.5},
           {"scale": -0.5}, {"lf_factor": 0.0}, {"lf_factor": 0.25}, {"degree": 3}, {"n_el": (3, 2, 1)},
           {"length": (1.0, 0.7, 1.2)}]


def in_new_thread(fn):
    out = []
    t = threading.Thread(target=lambda: out.append(fn()))
    t.start()
    t.join()
    return out[0]


@pytest.mark.parametrize("dtype", [torch.float64, torch.float32])
@pytest.mark.parametrize("op", ["laplace", "helmholtz", "convective", "vjp", "projection"])
def test_calls_do_not_depend_on_earlier_ones(op, dtype):
    gen = torch.Generator().manual_seed(11)
    calls = []
    for ch in CHANGES:
        a = {**BASE, **ch}
        desc = dgmf.make_desc(a.pop("degree"), a.pop("n_el"), a.pop("length"), **a)
        nel = desc.n_el[0] * desc.n_el[1] * desc.n_el[2]
        u, w = (torch.rand(3, nel, (desc.degree + 1) ** 3, generator=gen, dtype=torch.float64).to("cuda", dtype)
                for _ in range(2))
        tau = torch.rand(nel, generator=gen, dtype=torch.float64).to("cuda", dtype)
        if op == "helmholtz":   # also the mass factor alone changes
            for m in (0.0, 2.0):
                calls.append(lambda d=desc, u=u, m=m: dgmf.apply_helmholtz(d, u, m))
        else:
            calls.append({"laplace": lambda d=desc, u=u: dgmf.apply_laplace(d, u),
                          "convective": lambda d=desc, u=u: dgmf.apply_convective(d, u),
                          "vjp": lambda d=desc, u=u, w=w: dgmf.vjp_convective(d, u, w),
                          "projection": lambda d=desc, u=u, t=tau: dgmf.apply_projection(d, u, t, t)}[op])
    want = [in_new_thread(c) for c in calls]
    for _ in range(2):
        for i in list(range(len(calls))) + [0, 3, 0, 3]:
            assert torch.equal(calls[i](), want[i]), i


def test_bound_arguments_are_checked_as_before():
    desc = dgmf.make_desc(2, (2, 2, 2), n_comp=3)
    u = torch.rand(3, 8, 27, device="cuda", dtype=torch.float64)
    dgmf.apply_convective(desc, u)
    for bad, err in ((u[:, :4], ValueError), (u.float().double()[:, :, ::2], ValueError),
                     (u.to(torch.float16), TypeError), (u.cpu(), ValueError)):
        with pytest.raises(err):
            dgmf.apply_convective(desc, bad)
    with pytest.raises((ValueError, TypeError)):
        dgmf.apply_convective(desc, u, out=u.float())
    with pytest.raises(AttributeError):   # None has no shape
        dgmf.vjp_convective(desc, u, None)
    with pytest.raises(AttributeError):   # None has no shape
        dgmf.apply_projection(desc, u, None, None)
