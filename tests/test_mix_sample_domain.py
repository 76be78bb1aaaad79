"""Channel mixing in the sample domain (equal degrees 1..8, C1 C2 >= 128, Co <=
128; the plans' hook takes it at the small sizes of these tests too): every degree, channel counts about the 16 and 32 of the operand tiles, in
both roles of the two inputs, output channels about the 16 and 32 of a
workgroup, batches that leave the last workgroup of the low degrees short.

Tolerance.  Per output row |y - y64| <= 1e-6 sum_p |W_p| |T_p|: operands in
three bf16 parts hold fp32 values exactly, products leave out 2^-24 of a term at
worst, and the four sums of a result (samples, over c1, over c2, analysis) round
at 2^-24 of their partial sums, a handful of times each: about ten times 2^-24,
6e-7, were they to add up (seen: 1e-7, as for the fp32 pair products)."""
import os

import numpy as np
import pytest

torch = pytest.importorskip("torch")

from oracle import gtp_oracle as O  # noqa: E402
from paper_2401_10216_amd import gtp  # noqa: E402

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True)
def _sampled(monkeypatch):
    monkeypatch.setenv("GTP_TEST_MIX", "sampled")


def _products(L, x1, x2):
    B, C1, K = x1.shape
    C2 = x2.shape[1]
    a = np.repeat(x1[:, :, None], C2, 2).reshape(-1, K)
    b = np.repeat(x2[:, None], C1, 1).reshape(-1, K)
    return O.gtp(a, b, L, L, L).reshape(B, C1 * C2, K)


def _check(L, x1, x2, W, tol=1e-6):
    """Row by row against the oracle's pair products, in units of the terms."""
    y = gtp.gtp_channel_mix(gtp.Plan(L, L, L), x1.cuda(), x2.cuda(), W.cuda())
    T = _products(L, x1.double().numpy(), x2.double().numpy())
    w = W.double().numpy().reshape(W.shape[0], -1)
    ref = np.einsum("op,bpk->bok", w, T)
    bound = np.einsum("op,bp->bo", np.abs(w), np.linalg.norm(T, axis=2))
    err = np.linalg.norm(y.cpu().numpy().astype(np.float64) - ref, axis=2)
    assert (err <= tol * bound).all(), (L, (err / np.maximum(bound, 1e-300)).max())


@pytest.mark.parametrize("L", range(1, 9))
@pytest.mark.parametrize("B,C1,C2,Co,dt", [(1, 2, 64, 1, torch.float32), (5, 16, 8, 16, torch.float32),
                                           (3, 17, 33, 17, torch.bfloat16), (2, 33, 4, 33, torch.float32),
                                           (5, 40, 65, 2, torch.float32), (2, 12, 11, 128, torch.bfloat16)])
def test_sizes(L, B, C1, C2, Co, dt):
    g = torch.Generator().manual_seed(1000 * L + C1)
    x1, x2 = (torch.randn((B, c, (L + 1) ** 2), generator=g).to(dt) for c in (C1, C2))
    _check(L, x1, x2, torch.randn((Co, C1, C2), generator=g))


@pytest.mark.parametrize("L", [1, 4, 6, 8])
def test_channel_scales(L):
    """Channels over many orders of magnitude, every output weighing one pair:
    each row holds to its own size, in either input's role."""
    g = torch.Generator().manual_seed(L)
    n = 20
    x1, x2 = (torch.randn((3, n, (L + 1) ** 2), generator=g) for _ in range(2))
    x1 = x1 * torch.logspace(-12, 6, n)[None, :, None]
    x2 = x2 * torch.logspace(8, -9, n)[None, :, None]
    W = torch.zeros((n, n, n))
    for i in range(n):
        W[i, i, i] = 10.0 ** (i - 8)
    _check(L, x1, x2, W)
    _check(L, x2, x1, W)
    x1[1] = 0.0  # an entry of zeros, and a channel of zeros
    x2[2, 5] = 0.0
    _check(L, x1, x2, W)


def _roles(x1, x2, W):
    """The call, and the same with the two inputs' roles exchanged."""
    return (x1, x2, W), (x2, x1, W.transpose(1, 2).contiguous())


@pytest.mark.parametrize("L", [1, 2, 4, 6, 8])
@pytest.mark.parametrize("n", [16, 33])
@pytest.mark.parametrize("s", [1e-6, 1e-12, 1e-30])
def test_outputs_of_any_size(L, n, s):
    """Half of one input's channels s times smaller, each output weighing one
    of them (all of the other input's): outputs of one tile lie s apart, and
    each holds to its own terms."""
    g = torch.Generator().manual_seed(L)
    x1, x2 = (torch.randn((3, n, (L + 1) ** 2), generator=g) for _ in range(2))
    x1[:, n // 2:] *= s
    W = torch.zeros((n, n, n))
    for i in range(n):
        W[i, i] = torch.randn(n, generator=g)
    for call in _roles(x1, x2, W):
        _check(L, *call)


@pytest.mark.parametrize("L", [1, 2, 4, 6, 8])
@pytest.mark.parametrize("n", [16, 33])
@pytest.mark.parametrize("s", [1e-6, 1e-9, 1e-12, 1e-30])
def test_weights_of_any_size(L, n, s):
    """Weights s times the others: where they meet a channel 1 / s times larger
    (all terms alike), and where the heavy ones meet a channel of zeros."""
    g = torch.Generator().manual_seed(L)
    x1, x2 = (torch.randn((3, n, (L + 1) ** 2), generator=g) for _ in range(2))
    W = torch.randn((n, n, n), generator=g)
    big, light = x1.clone(), W.clone()
    big[:, 3] /= s
    light[:, 3] *= s
    dead, heavy = x1.clone(), W.clone()
    dead[:, 3] = 0.0
    heavy[:, 3] /= s
    for call in (*_roles(big, x2, light), *_roles(dead, x2, heavy)):
        _check(L, *call)


@pytest.mark.parametrize("L", [1, 6])
def test_inputs_over_the_exponent_range(L):
    """One entry's channels 1e40 apart, and entries and weights near the ends of
    fp32's range whose products lie within it."""
    g = torch.Generator().manual_seed(L)
    x1, x2 = (torch.randn((4, 16, (L + 1) ** 2), generator=g) for _ in range(2))
    x1[0, :8] *= 1e18
    x1[0, 8:] *= 1e-22
    x1[1] *= 1e30
    x2[1] *= 1e-25
    x1[2] *= 1e-30
    x2[2] *= 1e20
    W = torch.zeros((16, 16, 16))
    for i in range(16):
        W[i, i] = torch.randn(16, generator=g)
    W[5] *= 1e15
    W[6] *= 1e-20
    for call in _roles(x1, x2, W):
        _check(L, *call)


@pytest.mark.parametrize("L", [1, 2, 6])
def test_not_finite_stays_in_its_entry(L):
    g = torch.Generator().manual_seed(L)
    x1, x2 = (torch.randn((6, 16, (L + 1) ** 2), generator=g).cuda() for _ in range(2))
    W = torch.randn((4, 16, 16), generator=g).cuda()
    plan = gtp.Plan(L, L, L)
    want = gtp.gtp_channel_mix(plan, x1, x2, W)
    x1[1, 3, 0] = float("nan")
    x2[4, 15, 1] = float("inf")
    got = gtp.gtp_channel_mix(plan, x1, x2, W)
    for b in range(6):
        if b in (1, 4):
            assert not torch.isfinite(got[b]).any(), b
        else:
            assert torch.equal(got[b], want[b]), b


@pytest.mark.parametrize("L", [1, 2, 6])
@pytest.mark.parametrize("C1,C2", [(16, 8), (8, 16), (40, 33), (33, 40)])
@pytest.mark.parametrize("which", [0, 1])
def test_channels_without_a_finite_value(L, C1, C2, which):
    """A channel of NaN, and one of a single Inf among zeros, beside ordinary
    ones, in either input and either role, one and several tiles of channels:
    none of the entry's outputs is a number, the other entries' are unchanged."""
    g = torch.Generator().manual_seed(L)
    x = [torch.randn((6, c, (L + 1) ** 2), generator=g).cuda() for c in (C1, C2)]
    W = torch.randn((4, C1, C2), generator=g).cuda()
    plan = gtp.Plan(L, L, L)
    want = gtp.gtp_channel_mix(plan, *x, W)
    x[which][1, 3] = float("nan")
    x[which][4, 5] = 0.0
    x[which][4, 5, 0] = float("inf")
    got = gtp.gtp_channel_mix(plan, *x, W)
    for b in range(6):
        if b in (1, 4):
            assert not torch.isfinite(got[b]).any(), b
        else:
            assert torch.equal(got[b], want[b]), b


@pytest.mark.parametrize("L,B,C1,C2,Co", [(6, 512, 32, 32, 32), (1, 8192, 24, 24, 8), (8, 16, 32, 32, 32)])
def test_the_way_that_pays_is_taken(monkeypatch, L, B, C1, C2, Co):
    """At sizes where the sample domain pays, a plan without the hook gives its results, bit for bit."""
    g = torch.Generator(device="cuda").manual_seed(L)
    x1, x2 = (torch.randn((B, c, (L + 1) ** 2), generator=g, device="cuda") for c in (C1, C2))
    W = torch.randn((Co, C1, C2), generator=g, device="cuda")
    hooked = gtp.gtp_channel_mix(gtp.Plan(L, L, L), x1, x2, W)
    monkeypatch.delenv("GTP_TEST_MIX")
    assert torch.equal(gtp.gtp_channel_mix(gtp.Plan(L, L, L), x1, x2, W), hooked)


@pytest.mark.parametrize("L", range(1, 9))
@pytest.mark.parametrize("B,C1,C2,Co,dt", [(5, 16, 12, 16, torch.float32), (3, 40, 9, 33, torch.bfloat16),
                                           (6, 17, 33, 17, torch.float32)])
def test_reads_no_lds_it_has_not_written(L, B, C1, C2, Co, dt):
    """The same bits from the build whose kernels fill their LDS with NaN first."""
    g = torch.Generator().manual_seed(L)
    x1, x2 = (torch.randn((B, c, (L + 1) ** 2), generator=g).to(dt).cuda() for c in (C1, C2))
    W = torch.randn((Co, C1, C2), generator=g).cuda()
    y = gtp.gtp_channel_mix(gtp.Plan(L, L, L), x1, x2, W)
    with gtp.use_library(os.path.join(os.path.dirname(gtp.__file__), "libgtp_poison.so")):
        z = gtp.gtp_channel_mix(gtp.Plan(L, L, L), x1, x2, W)
        torch.cuda.synchronize()
    assert torch.isfinite(y).all() and torch.equal(y, z)


@pytest.mark.parametrize("L,C1,C2,Co", [(1, 33, 20, 17), (6, 32, 32, 32), (8, 16, 40, 5)])
def test_several_streams(L, C1, C2, Co):
    """Calls on four streams at once, each with its own inputs: the results of one after the other."""
    g = torch.Generator(device="cuda").manual_seed(L)
    plan = gtp.Plan(L, L, L)
    jobs = [[torch.randn(s, generator=g, device="cuda") for s in ((37, C1, (L + 1) ** 2), (37, C2, (L + 1) ** 2),
                                                                 (Co, C1, C2))] for _ in range(4)]
    want = [gtp.gtp_channel_mix(plan, *j) for j in jobs]
    streams = [torch.cuda.Stream() for _ in jobs]
    torch.cuda.synchronize()
    got = []
    for _ in range(5):
        for s, j in zip(streams, jobs):
            with torch.cuda.stream(s):
                got.append(gtp.gtp_channel_mix(plan, *j))
    torch.cuda.synchronize()
    for i, y in enumerate(got):
        assert torch.equal(y, want[i % 4]), i
