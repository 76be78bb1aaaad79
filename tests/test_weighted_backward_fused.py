"""The one-kernel backward of the weighted product (equal degrees 1..8): every
degree, channel counts about the 64 lanes of a wave (a lane keeps one weight
row), batches of one and several passes of the grid, subsets of the gradients.

Tolerances.  Rows of dx as in the other fp32 product tests: 1e-5 of the row's
norm (these kernels show 3e-7 per coefficient).  A weight gradient is a sum
over products of dot products <a, u> on one degree's 2 l + 1 coefficients: an
error of 3e-7 |u| per coefficient of u gives at most 3e-7 sqrt(2 l + 1) |a_l|
|u| <= 1.3e-6 |a_l| |u| per product, and the fp32 sums add less; so 2e-6 of the
sum of |a_l| |u| over the row's products is allowed."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from oracle import gtp_oracle as O  # noqa: E402
from paper_2401_10216_amd import gtp  # noqa: E402

pytestmark = pytest.mark.gpu


def _reference(L, x1, x2, dy, w1, w2, wo, per_channel):
    """fp64 gradients and the weight gradients' error scales, from the oracle's products."""
    B, C, K = x1.shape
    deg = O.degree_index(L)

    def prod(a, b):
        return O.gtp(a.reshape(-1, K), b.reshape(-1, K), L, L, L).reshape(B, C, K)

    W1, W2, WO = w1[:, deg], w2[:, deg], wo[:, deg]
    z, u1, u2 = prod(W1 * x1, W2 * x2), prod(WO * dy, W2 * x2), prod(WO * dy, W1 * x1)

    def rows(a, u):
        s, m = np.zeros((C, L + 1)), np.zeros((C, L + 1))
        for l in range(L + 1):
            s[:, l] = (a * u)[:, :, deg == l].sum((0, 2))
            m[:, l] = (np.linalg.norm(a[:, :, deg == l], axis=2) * np.linalg.norm(u, axis=2)).sum(0)
        return (s, m) if per_channel else (s.sum(0, keepdims=True), m.sum(0, keepdims=True))

    return {"dx1": W1 * u1, "dx2": W2 * u2, "dw1": rows(x1, u1), "dw2": rows(x2, u2), "dwout": rows(dy, z)}


@pytest.mark.parametrize("L", range(1, 9))
@pytest.mark.parametrize("B,C,per_channel,dt", [(1, 1, True, torch.float32), (7, 63, True, torch.float32),
                                                (9, 65, True, torch.bfloat16), (3, 96, False, torch.bfloat16),
                                                (130, 2, True, torch.float32), (1, 257, False, torch.float32)])
def test_all_gradients(L, B, C, per_channel, dt):
    g = torch.Generator().manual_seed(100 * L + C)
    K, R = (L + 1) ** 2, C if per_channel else 1
    x1, x2 = (torch.randn((B, C, K), generator=g).to(dt) for _ in range(2))
    dy = torch.randn((B, C, K), generator=g)
    w1, w2, wo = (1 + 0.5 * torch.randn((R, L + 1), generator=g) for _ in range(3))
    plan = gtp.Plan(L, L, L)
    dev = [t.cuda() for t in (x1, x2, dy, w1, w2, wo)]
    got = gtp.gtp_full_weighted_backward(plan, *dev, per_channel=per_channel)
    again = gtp.gtp_full_weighted_backward(plan, *dev, per_channel=per_channel)
    ref = _reference(L, *(t.double().numpy() for t in (x1, x2, dy, w1, w2, wo)), per_channel)
    for k, v in got.items():
        assert torch.equal(v, again[k]), k  # deterministic
        v = v.cpu().numpy().astype(np.float64)
        if k.startswith("dx"):
            err = O.max_rel_err(v.reshape(-1, K), ref[k].reshape(-1, K))
        else:
            err = float((np.abs(v - ref[k][0]) / ref[k][1]).max())
        print(L, B, C, per_channel, dt, k, f"err={err:.2e}", flush=True)
        assert err <= (1e-5 if k.startswith("dx") else 2e-6), (k, err)
    # a gradient alone is the same; one weight left out stands for ones
    for k in got:
        alone = gtp.gtp_full_weighted_backward(plan, *dev, per_channel=per_channel, need=(k,))
        assert torch.equal(alone[k], got[k]), k
    ones = gtp.gtp_full_weighted_backward(plan, dev[0], dev[1], dev[2], None, torch.ones_like(dev[4]), None,
                                          per_channel=per_channel)
    none = gtp.gtp_full_weighted_backward(plan, dev[0], dev[1], dev[2], per_channel=per_channel)
    for k in got:
        assert torch.equal(ones[k], none[k]), k


def test_several_passes_of_the_grid():
    """More products than lanes: 2048 waves take one pass of 131072, the rows' sums go on over the passes."""
    L, B, C = 1, 3001, 96
    g = torch.Generator(device="cuda").manual_seed(5)
    x1, x2, dy = (torch.randn((B, C, 4), generator=g, device="cuda") for _ in range(3))
    w = [1 + 0.5 * torch.randn((C, 2), generator=g, device="cuda") for _ in range(3)]
    got = gtp.gtp_full_weighted_backward(gtp.Plan(L, L, L), x1, x2, dy, *w, per_channel=True)
    ref = _reference(L, *(t.double().cpu().numpy() for t in (x1, x2, dy, *w)), True)
    for k in ("dw1", "dw2", "dwout"):
        err = float((np.abs(got[k].cpu().numpy() - ref[k][0]) / ref[k][1]).max())
        assert err <= 2e-6, (k, err)
    for k in ("dx1", "dx2"):
        # over all rows at once: among 288096 rows some cancel to where their own norm is no measure
        d = got[k].cpu().numpy() - ref[k]
        assert np.linalg.norm(d) <= 1e-6 * np.linalg.norm(ref[k])
