"""The torch.autograd wrapper of the adjoint: its gradients equal those of the direct C-ABI
calls bitwise, and match central finite differences of the FP64 oracle."""
import numpy as np
import pytest
import torch

import oracle
from paper_1808_08555_amd import inputs, lbm3
from paper_1808_08555_amd.autograd import ternary_run

pytestmark = pytest.mark.gpu

SIGMA = (0.006, 0.010, 0.012)
TAU = (0.7, 0.8, 0.9)


def _janus(nx, ny, R):
    y, x = np.mgrid[0:ny, 0:nx].astype(float)
    inside = (x - nx / 2) ** 2 + (y - ny / 2) ** 2 <= R * R
    lab = np.full((ny, nx), 2)
    lab[inside & (x < nx / 2)] = 0
    lab[inside & (x >= nx / 2)] = 1
    return inputs.rho_from_labels(lab), lab


@pytest.mark.parametrize("device", ["cpu", "cuda"])
def test_autograd_equals_direct_adjoint(device):
    nx, ny, steps, every = 24, 20, 12, 4
    rho0, _ = _janus(nx, ny, 6.0)
    target = inputs.loss_target(rho0[0], seed=5550)
    s = torch.tensor(SIGMA, dtype=torch.float64, device=device, requires_grad=True)
    r = torch.tensor(rho0, dtype=torch.float64, device=device, requires_grad=True)
    out = ternary_run(s, r, steps, every, tau=TAU)
    assert out.device.type == device and out.shape == (ny, nx)
    loss = ((out - torch.tensor(target, device=device)) ** 2).sum()
    loss.backward()
    L = lbm3.Lattice(nx, ny, SIGMA, TAU).init(rho0)
    lbm3.lbm3_adjoint_record(L.h, steps, every)
    rho_T = L.densities()
    ds, dr = lbm3.lbm3_adjoint(L.h, 2.0 * (rho_T[0] - target), nx, ny)
    L.close()
    assert np.array_equal(out.detach().cpu().numpy(), rho_T[0])
    assert np.array_equal(s.grad.cpu().numpy(), ds)
    assert np.array_equal(r.grad.cpu().numpy(), dr)
    assert s.grad.device.type == device and r.grad.device.type == device


def test_autograd_sigma_gradient_matches_oracle_differences():
    """A loss that is not quadratic (weighted sum of rho_1(T)), so the upstream gradient is
    a fixed field rather than a residual."""
    nx, ny, steps, h = 20, 18, 8, 1e-6
    rho0, _ = _janus(nx, ny, 5.0)
    wts = inputs.loss_target(np.zeros((ny, nx)), seed=11)
    s = torch.tensor(SIGMA, dtype=torch.float64, requires_grad=True)
    out = ternary_run(s, torch.tensor(rho0), steps, 2, tau=TAU)
    (out * torch.tensor(wts)).sum().backward()

    def L(sig):
        p = oracle.Params(nx, ny, tuple(sig), TAU)
        return float((oracle.density(oracle.run(p, oracle.init(p, rho0), steps))[0] * wts).sum())

    for q in range(3):
        sp, sm = list(SIGMA), list(SIGMA)
        sp[q] += h
        sm[q] -= h
        fd = (L(sp) - L(sm)) / (2 * h)
        print(f"dL/dsigma[{q}] autograd {s.grad[q].item():.10e} fd {fd:.10e}")
        assert abs(s.grad[q].item() - fd) <= 1e-5 * max(1e-3, abs(fd))


def test_autograd_second_backward_raises():
    rho0, _ = _janus(12, 12, 3.0)
    s = torch.tensor(SIGMA, dtype=torch.float64, requires_grad=True)
    out = ternary_run(s, torch.tensor(rho0), 4, 2)
    out.sum().backward(retain_graph=True)
    with pytest.raises(RuntimeError):
        out.sum().backward()


def test_repeated_gradients_reuse_workspaces_and_stay_equal():
    """Workspaces kept from one run for the next: gradients of different sizes and inputs in
    turn, on two streams and from two threads at once, equal those of runs that had to
    allocate (bit for bit), also after the kept memory was given back."""
    import threading
    sigma = torch.tensor([0.006, 0.010, 0.012], dtype=torch.float64)

    def grad(n, seed, steps):
        rho = torch.from_numpy(np.ascontiguousarray(_janus(n, n + 5, n / 6 + seed)[0]))
        s, r = sigma.clone().requires_grad_(), rho.requires_grad_()
        out = ternary_run(s, r, steps, ckpt_every=4, tau=(0.8, 0.8, 0.8))
        return [x.clone() for x in torch.autograd.grad((out ** 2).sum(), (s, r))]

    cases = [(96, 1, 12), (128, 2, 8), (96, 3, 12), (128, 2, 8)]
    fresh = []
    for c in cases:
        lbm3.lbm3_release_cached()
        fresh.append(grad(*c))
    for got, want in zip([grad(*c) for c in cases], fresh):
        assert all(torch.equal(a, b) for a, b in zip(got, want))
    both = [None, None]

    def work(k):
        with torch.cuda.stream(torch.cuda.Stream()):
            both[k] = [grad(*c) for c in cases]

    ts = [threading.Thread(target=work, args=(k,)) for k in (0, 1)]
    for t in ts:
        t.start()
    for t in ts:
        t.join()
    for r in both:
        for got, want in zip(r, fresh):
            assert all(torch.equal(a, b) for a, b in zip(got, want))
    lbm3.lbm3_release_cached()
