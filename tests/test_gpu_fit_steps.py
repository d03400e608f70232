"""The fit's step kernels (``csrc/saf_fit_kernels.h``) at the edges of their
32-entry blocks, 1024-entry tiles and distance chunks (every chunk size is
reached by some head count and length below), against float64.

One step from the fit's start moves each parameter by
``lr g / (|g| + eps)`` (Adam's first step), a sign wherever |g| >> eps; the
float32 gradient g = (marginal - eta) / T carries the rounding of sums of at
most T terms, so where |g| is well above that rounding the step must be the
float64 one.  Two steps then depend on the size of both gradients.
Parameters are compared where the float64 gradient of both steps exceeds
1e-3 of the largest, to 1e-3 of the learning rate per step.

``floor`` 1e-30 with a target whose offset 0 and early columns are (almost)
empty gives rows whose normaliser lies below exp(-40) of the head's largest
factors: the entry-by-entry path of both kernels.
"""

import numpy as np
import pytest

from gpu_helpers import announce, torch_cuda

pytestmark = pytest.mark.gpu

LR = 0.05


def _logits(a, r):
    T = a.size
    off = np.arange(T)[:, None] - np.arange(T)[None, :]
    return np.where(off >= 0, a[None, :] + r[np.clip(off, 0, None)], -np.inf), off


def _steps(ea, er, floor, steps):
    """Float64 fit; returns a, r, log Z and the gradients of each step."""
    T = ea.size
    a, r = np.zeros(T), np.log(np.maximum(er / (T - np.arange(T)), floor))
    m, v, grads = np.zeros((2, T)), np.zeros((2, T)), []
    for t in range(1, steps + 2):
        L, off = _logits(a, r)
        top = L.max(1, keepdims=True)
        z = top[:, 0] + np.log(np.exp(L - top).sum(1))
        if t > steps:
            return a, r, z, grads
        P = np.exp(L - z[:, None])
        dia = np.bincount(np.clip(off, 0, None).ravel(), weights=P.ravel(), minlength=T)
        g = np.stack([P.sum(0) - ea, dia - er]) / T
        grads.append(g)
        m, v = 0.9 * m + 0.1 * g, 0.999 * v + 0.001 * g * g
        d = LR * (m / (1 - 0.9 ** t)) / (np.sqrt(v / (1 - 0.999 ** t)) + 1e-8)
        a, r = a - d[0], r - d[1]


@pytest.mark.parametrize("H,T,low", [(1, 1, False), (2, 31, False), (2, 33, False), (1, 127, True), (3, 257, False),
                                     (2, 1000, True), (2, 1023, False), (2, 1025, False), (64, 513, False),
                                     (16, 2080, False)])
def test_fit_steps_match_float64(H, T, low):
    torch = torch_cuda()
    from paper_2609_34650_amd import binding
    announce(f"fit steps H={H} T={T} low={low}")
    g = np.random.Generator(np.random.PCG64(77 + T))
    i, floor = np.arange(T), 1e-30 if low else 1e-9
    # Marginals of a random pattern's scale: non-negative, each summing to T.
    ea, er = (g.random((H, T)) ** 3 * (T - i) / T + 1e-6 for _ in range(2))
    if low:
        er[:, : T // 8] = 0.0   # the first offsets are (almost) never used
    ea, er = (x * (T / x.sum(1, keepdims=True)) for x in (ea, er))
    ea, er = ea.astype(np.float32), er.astype(np.float32)
    dev = [torch.from_numpy(x).to("cuda") for x in (ea, er)]
    ne = torch.zeros(H, dtype=torch.float64, device="cuda")
    a, r, z, _ = binding.saf_compact_fit(*dev, ne, steps=2, lr=LR, floor_value=floor)
    torch.cuda.synchronize()
    for h in sorted({0, H // 2, H - 1}):
        oa, orr, oz, grads = _steps(ea[h].astype(np.float64), er[h].astype(np.float64), floor, 2)
        big = np.ones((2, T), bool)
        for gr in grads:
            big &= np.abs(gr) > max(1e-3 * np.abs(gr).max(), 1e-7)
        for got, want, sel in ((a, oa, big[0]), (r, orr, big[1])):
            got = got[h].double().cpu().numpy()
            assert np.isfinite(got).all()
            np.testing.assert_allclose(got[sel], want[sel], rtol=1e-6, atol=2e-3 * LR)
        # log Z at the GPU's own parameters
        L, _ = _logits(a[h].double().cpu().numpy(), r[h].double().cpu().numpy())
        top = L.max(1, keepdims=True)
        np.testing.assert_allclose(z[h].double().cpu().numpy(), top[:, 0] + np.log(np.exp(L - top).sum(1)),
                                   rtol=2e-6, atol=2e-5)
