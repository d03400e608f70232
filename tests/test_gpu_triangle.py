"""The one-pass triangle sums (``csrc/saf_tri.h``) at the edges of their
256 x 256 blocks, 64-row wavefront chunks and 8-row load steps, against numpy
in float64: target marginals (``saf_fit_targets``) and the finalisation's
marginals and entropy part (``saf_calib_finalize``).

Entries above the diagonal are NaN: they are never to be read into a sum.
Bars: float32 sums of n non-negative terms in any order differ from the exact
sum by less than n 2^-24 of it; n <= T here, and a handful of roundings per
term (floor, 1 / s, log) come on top.
"""

import numpy as np
import pytest

from gpu_helpers import announce, torch_cuda

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("T", [1, 7, 8, 63, 64, 65, 255, 256, 257, 321, 513, 777])
def test_triangle_sums_match_numpy(T):
    torch = torch_cuda()
    from paper_2609_34650_amd import binding
    announce(f"triangle sums T={T}")
    H = 2
    g = np.random.Generator(np.random.PCG64(1000 + T))
    mean = np.tril(g.random((H, T, T), dtype=np.float32) ** 4 / T)
    mean[:, T // 2, : T // 2 + 1] = 0.0  # zeros: floored by the targets, no entropy in the finalisation
    stored = np.where(np.tril(np.ones((T, T), bool))[None], mean, np.float32(np.nan))
    dev = torch.from_numpy(stored).to("cuda")
    rtol = (T + 16) * 2.0 ** -24

    def sums(P):
        return P.sum(0), np.array([np.trace(P, -d) for d in range(T)])

    state = binding.CalibState(H, T, "cuda")
    state.mean.copy_(dev)
    state.stats.zero_()
    state.n_seen = 3
    out = binding.saf_calib_finalize(state)
    ea, er, ne = binding.saf_fit_targets(dev)
    torch.cuda.synchronize()
    for h in range(H):
        m = mean[h].astype(np.float64)
        col, dia = sums(m)
        np.testing.assert_allclose(out["eta_abs"][h].double().cpu().numpy(), col, rtol=rtol, atol=0)
        np.testing.assert_allclose(out["eta_rel"][h].double().cpu().numpy(), dia, rtol=rtol, atol=0)
        ent = -np.sum(m[m > 0] * np.log(m[m > 0])) / T  # s_KL of a state whose sums are 0
        np.testing.assert_allclose(float(out["s_kl"][h]), ent, rtol=2e-6, atol=0)
        Pi = np.tril(np.maximum(m, 1e-9))
        Pi /= Pi.sum(1, keepdims=True)
        col, dia = sums(Pi)
        np.testing.assert_allclose(ea[h].double().cpu().numpy(), col, rtol=2 * rtol, atol=0)
        np.testing.assert_allclose(er[h].double().cpu().numpy(), dia, rtol=2 * rtol, atol=0)
        P = Pi[Pi > 0]
        np.testing.assert_allclose(float(ne[h]), np.sum(P * np.log(P)), rtol=2e-6, atol=1e-9)
