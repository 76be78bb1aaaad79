"""Channel mixing by pair products from 128 pairs on (k_mix_fused, shapes of few
channels against many; the plans' hook takes it at every shape here): the error
of its sums over the pairs."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from oracle import gtp_oracle as O  # noqa: E402
from paper_2401_10216_amd import gtp  # noqa: E402

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("L", [1, 2, 4, 6, 8])
@pytest.mark.parametrize("C1,C2,Co,dt", [(4, 32, 16, torch.float32), (32, 4, 33, torch.bfloat16), (5, 41, 8, torch.float32),
                                         (128, 4, 64, torch.float32), (4, 256, 100, torch.float32)])
def test_error_does_not_grow_with_the_pairs(monkeypatch, L, C1, C2, Co, dt):
    """2-norm error against 64 bits.  A product errs by 1.2e-7 of itself at most
    of these degrees, the sum over them, in runs of 32 pairs, 256 and all,
    rounds at sqrt(8 + 8 + 4) 2^-25 of its size and less: 1.8e-7 together.  1.9e-7
    allowed (one sum in order: 2.2e-7 at 128 pairs to 5.8e-7 at 1024)."""
    monkeypatch.setenv("GTP_TEST_MIX", "pairs")
    g = torch.Generator().manual_seed(10 * L + C1)
    B, K = 8, (L + 1) ** 2
    x1, x2 = (torch.randn((B, c, K), generator=g).to(dt) for c in (C1, C2))
    W = torch.randn((Co, C1, C2), generator=g) / (C1 * C2) ** 0.5
    y = gtp.gtp_channel_mix(gtp.Plan(L, L, L), x1.cuda(), x2.cuda(), W.cuda()).cpu().double().numpy()
    a = np.repeat(x1.double().numpy()[:, :, None], C2, 2).reshape(-1, K)
    b = np.repeat(x2.double().numpy()[:, None], C1, 1).reshape(-1, K)
    T = O.gtp(a, b, L, L, L).reshape(B, C1 * C2, K)
    ref = np.einsum("op,bpk->bok", W.double().numpy().reshape(Co, -1), T)
    err = np.linalg.norm(y - ref) / np.linalg.norm(ref)
    print(L, (C1, C2, Co), dt, f"{err:.3e}", flush=True)
    assert err <= 1.9e-7, err
