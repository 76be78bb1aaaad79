"""The split-operand matrix-core product kernel (degrees 16, 32 and every
triple padded to them): its operand and index images on the CPU, and the
kernel at the sizes and values where it can go wrong on the GPU."""
import os
import shutil
import subprocess

import numpy as np
import pytest

torch = pytest.importorskip("torch")

from oracle import gtp_oracle as O  # noqa: E402
from paper_2401_10216_amd import gtp  # noqa: E402

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2401_10216_amd", "csrc")


@pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")
def test_operand_and_index_images(tmp_path):
    exe = str(tmp_path / "mfma_host")
    r = subprocess.run(["g++", "-O1", "-std=c++17", f"-I{CSRC}", "-o", exe,
                        os.path.join(ROOT, "tests", "mfma_host_main.cpp"), os.path.join(CSRC, "gtp_mfma_tables.cpp"),
                        os.path.join(CSRC, "gtp_tables.cpp")], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    r = subprocess.run([exe], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0 and r.stdout.strip().endswith("ok"), r.stdout


def _check(L1, L2, Lout, a, b, offset=0, what=""):
    """gtp_full of rows a, b (values already of the call's type) against the oracle, per product."""
    n = a.shape[0]
    plan = gtp.Plan(L1, L2, Lout)

    def dev(x):  # `offset` elements off the allocation's alignment
        buf = torch.empty(x.numel() + offset, dtype=x.dtype, device="cuda")
        v = buf[offset:].view(n, 1, x.shape[-1])
        v.copy_(x.view(n, 1, -1))
        return v

    y = gtp.gtp_full(plan, dev(a), dev(b)).cpu().numpy().astype(np.float64)[:, 0]
    ref = O.gtp_grid(a.double().numpy(), b.double().numpy(), L1, L2, Lout)
    err = O.max_rel_err(y, ref)
    print(what, (L1, L2, Lout), n, f"err={err:.2e}", flush=True)
    assert err <= 1e-6, err  # fp32: worst errors of these kernels are 1e-7 of the output norm


@pytest.mark.gpu
@pytest.mark.parametrize("degrees", [(16, 16, 16), (32, 32, 32), (9, 9, 9), (17, 20, 25), (0, 16, 16), (10, 3, 7),
                                     (5, 6, 30), (31, 1, 32), (16, 16, 40)])
@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
def test_edges_of_groups_and_rows(degrees, dtype):
    """Batches about the four products of a group; rows off 16-byte (4-byte) alignment."""
    L1, L2, Lout = degrees
    g = torch.Generator().manual_seed(7)
    for n, offset in ((1, 0), (3, 1), (4, 0), (4, 1), (5, 0), (11, 2)):
        a = torch.randn((n, (L1 + 1) ** 2), generator=g).to(dtype)
        b = torch.randn((n, (L2 + 1) ** 2), generator=g).to(dtype)
        _check(L1, L2, Lout, a, b, offset, f"{dtype} n={n} offset={offset}")


@pytest.mark.gpu
@pytest.mark.parametrize("L", [16, 32])
def test_scales_and_special_values(L):
    """Magnitudes over the fp32 range, sparse and concentrated rows, zeros, and a row of NaN or Inf beside others."""
    K = (L + 1) ** 2
    g = torch.Generator().manual_seed(8)
    a, b = torch.randn((12, K), generator=g), torch.randn((12, K), generator=g)
    a[0] *= 1e25  # the sum of squares overflows
    b[0] *= 1e-25  # and underflows
    a[1] *= 1e-30
    b[1] *= 1e20
    a[2] = 0.0
    a[2, K - 1] = 3.0  # single coefficients
    b[3] = 0.0
    b[3, 0] = -2.0
    a[4] = torch.as_tensor(O.real_sh(L, np.array([0.3]), np.array([1.1]))[0]) if hasattr(O, "real_sh") else a[4]
    b[4] = a[4]  # concentrated at one direction: the largest products the scales allow for
    a[5, L * L:] = 0.0
    b[6, : L * L] = 0.0
    a[7] *= 1e-12
    _check(L, L, L, a, b, 0, "scales")
    a[8] = 0.0
    a[9, 5] = float("nan")
    b[10, 7] = float("inf")
    y = gtp.gtp_full(gtp.Plan(L, L, L), a.cuda().view(12, 1, K), b.cuda().view(12, 1, K)).cpu()[:, 0]
    assert (y[8] == 0).all()
    assert y[9].isnan().any() and not y[10].isfinite().all()
    ok = [0, 1, 2, 3, 4, 5, 6, 7, 11]  # the same group's other rows are untouched
    ref = O.gtp_grid(a[ok].double().numpy(), b[ok].double().numpy(), L, L, L)
    assert O.max_rel_err(y[ok].numpy().astype(np.float64), ref) <= 1e-6


@pytest.mark.gpu
@pytest.mark.parametrize("degrees,bound", [((9, 9, 9), 1.05e-7), ((12, 12, 12), 1.18e-7), ((16, 16, 16), 1.35e-7),
                                           ((12, 12, 5), 1.065e-7), ((20, 20, 20), 1.31e-7), ((32, 32, 32), 1.67e-7)])
def test_error_no_larger_than_in_fp32(degrees, bound):
    """The 2-norm error over iid N(0, 1) products against 64 bits.  The bounds
    are what the fp32 pipeline (fp32 tables, operands and sums throughout)
    measures for the same; over these products they move by less than 0.5 %."""
    L1, L2, Lout = degrees
    g = torch.Generator().manual_seed(3)
    a, b = (torch.randn((2000 if Lout <= 16 else 400, (L + 1) ** 2), generator=g) for L in (L1, L2))
    y = gtp.gtp_full(gtp.Plan(L1, L2, Lout), a.cuda()[:, None], b.cuda()[:, None]).cpu().numpy()[:, 0].astype(np.float64)
    ref = O.gtp_grid(a.double().numpy(), b.double().numpy(), L1, L2, Lout)
    err = np.linalg.norm(y - ref) / np.linalg.norm(ref)
    print(degrees, f"{err:.3e}", flush=True)
    assert err <= bound, err


@pytest.mark.gpu
@pytest.mark.parametrize("degrees", [(12, 12, 12), (16, 16, 16), (32, 32, 32)])
def test_rows_of_zeros_and_of_vanishing_squares(degrees):
    """Zero rows of either input in every group of four, beside ordinary rows
    and rows whose squares vanish in fp32 (all of them, or all but one)."""
    L1, L2, Lout = degrees
    g = torch.Generator().manual_seed(9)
    a, b = (torch.randn((24, (L + 1) ** 2), generator=g) for L in (L1, L2))
    a[::4] = 0.0
    b[4:16:5] = 0.0
    a[5] *= 1e-25
    a[9] *= 1e-30
    b[9] *= 1e20
    b[13] *= 1e-25
    b[13, 3] = 1e-18
    a[17] *= 1e-28
    b[17] *= 1e-25  # the products stay above 1e-38 only where the factors' scales are taken out first
    a[17] *= 1e20
    y = gtp.gtp_full(gtp.Plan(L1, L2, Lout), a.cuda()[:, None], b.cuda()[:, None]).cpu().numpy()[:, 0].astype(np.float64)
    zero = (a == 0).all(1) | (b == 0).all(1)
    assert (y[zero.numpy()] == 0).all()
    ok = ~zero.numpy()
    ref = O.gtp_grid(a.double().numpy()[ok], b.double().numpy()[ok], L1, L2, Lout)
    assert O.max_rel_err(y[ok], ref) <= 1e-6


def _strided(x, offset):
    """x on the device, `offset` elements off the allocation's alignment."""
    buf = torch.empty(x.numel() + offset, dtype=x.dtype, device="cuda")
    v = buf[offset:].view(x.shape)
    v.copy_(x)
    return v


@pytest.mark.gpu
@pytest.mark.parametrize("degrees,n", [((16, 16, 16), 4 * 768 + 3), ((16, 16, 16), 4 * 1536 + 1), ((9, 12, 10), 4 * 768 + 2),
                                       ((32, 32, 32), 4 * 256 + 1), ((32, 32, 32), 4 * 512 + 3), ((17, 32, 20), 4 * 512 + 2)])
@pytest.mark.parametrize("types", [(torch.float32, torch.float32), (torch.bfloat16, torch.bfloat16),
                                   (torch.float32, torch.bfloat16)])
def test_later_turns_of_a_workgroup(degrees, n, types):
    """Batches past the 768 (degree 16) and 256 (32) workgroups' first groups:
    second and third turns, their short last group staged by element, rows on
    and off the loads' alignment; fp32 x bf16 as the gradient in x1.  Every row
    against the workgroup-per-product kernel, the first and last products of
    each turn against the oracle."""
    L1, L2, Lout = degrees
    g = torch.Generator().manual_seed(n)
    turn = 4 * (768 if max(degrees) <= 16 else 256)
    mixed = types[0] != types[1]
    if mixed:  # dx1 = P_L1(dy x2) of a plan (L1', L2, Lout') with Lout' = L1, L1' = Lout
        a = torch.randn((n, 1, (L1 + 1) ** 2), generator=g)
        b = torch.randn((n, 1, (L2 + 1) ** 2), generator=g).to(types[1])
    else:
        a, b = (torch.randn((n, 1, (L + 1) ** 2), generator=g).to(types[0]) for L in (L1, L2))
    for offset in (0, 1):
        ad, bd = _strided(a, offset), _strided(b, offset)

        def call(flags):
            if not mixed:
                return gtp.gtp_full(gtp.Plan(L1, L2, Lout, flags), ad, bd)
            x1 = torch.zeros((n, 1, (Lout + 1) ** 2), dtype=types[1], device="cuda")
            return gtp.gtp_full_backward(gtp.Plan(Lout, L2, L1, flags), x1, bd, ad, need_dx2=False)[0]

        y = call(0).cpu()[:, 0].double().numpy()
        ref = call(gtp.GTP_FORCE_GENERIC).cpu()[:, 0].double().numpy()
        assert O.max_rel_err(y, ref) <= 2e-6  # two kernels, each within 1e-6 of the oracle
        rows = sorted({r for t in range(0, n, turn) for r in (*range(t, t + 8), *range(t + turn - 8, t + turn))
                       if r < n} | set(range(n - 8, n)))
        exact = O.gtp_grid(a[rows, 0].double().numpy(), b[rows, 0].double().numpy(), L1, L2, Lout)
        assert O.max_rel_err(y[rows], exact) <= 1e-6


@pytest.mark.gpu
@pytest.mark.parametrize("L,B,C", [(16, 1039, 3), (32, 343, 3)])
def test_later_turns_with_channel_weights(L, B, C):
    """The same with weights per channel: three channels move through the groups of four."""
    K, deg = (L + 1) ** 2, O.degree_index(L)
    g = torch.Generator().manual_seed(L)
    a, b = (torch.randn((B, C, K), generator=g) for _ in range(2))
    w = [1 + 0.5 * torch.randn((C, L + 1), generator=g) for _ in range(3)]
    y = gtp.gtp_full_weighted(gtp.Plan(L, L, L), a.cuda(), b.cuda(), *(v.cuda() for v in w), per_channel=True).cpu().numpy()
    rows = [0, 1, 2, B // 2, B // 2 + 1, B - 3, B - 2, B - 1]
    x1, x2 = ((t[rows].double() * v.double()[:, deg]).numpy().reshape(-1, K) for t, v in ((a, w[0]), (b, w[1])))
    ref = O.gtp_grid(x1, x2, L, L, L) * np.tile(w[2].double().numpy()[:, deg], (len(rows), 1))
    assert O.max_rel_err(y[rows].reshape(-1, K).astype(np.float64), ref) <= 2e-6
    generic = gtp.gtp_full_weighted(gtp.Plan(L, L, L, gtp.GTP_FORCE_GENERIC), a.cuda(), b.cuda(), *(v.cuda() for v in w),
                                    per_channel=True).cpu().numpy()
    assert O.max_rel_err(y.reshape(-1, K).astype(np.float64), generic.reshape(-1, K).astype(np.float64)) <= 4e-6
