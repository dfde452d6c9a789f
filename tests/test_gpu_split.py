"""GPU parity where tiles and K slices have remainders: the likelihood pass's
recurrence and 128-row mixture tiles, which run on the bf16 matrix unit from
three-term splits, and the training gradient over rows that do not fill the
last slice, chunk or list of rows."""

import numpy as np
import pytest
import torch

import parity
from oracle import wm as owm
from paper_2205_01435_amd import _lib as wmlib
from paper_2205_01435_amd import workloads as wl
from test_gpu_grad import _case, _check

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def gpu():
    assert torch.cuda.is_available(), "GPU tests need a ROCm GPU"
    wmlib.load()
    yield


@pytest.mark.parametrize("seed,B,T,Z,H,A,K", [
    (31, 97, 23, 24, 272, 70, 8),   # 2231 rows: several slices, the last short of a chunk
    (32, 33, 31, 40, 144, 9, 5),    # 1023 rows; 192 and 592 product columns
    (33, 5, 3, 8, 16, 3, 1),        # fewer rows than one chunk
    (35, 50, 5, 24, 256, 6, 2),     # reverse steps in one launch; a short row block
    (36, 9, 3, 8, 320, 4, 1),       # ... with slices that end inside a stage of loads
    (34, 700, 25, 8, 16, 1, 1),     # one action: every row of a block in its list, a second block in each chunk
])
def test_grad_slices(seed, B, T, Z, H, A, K):
    ln = np.random.default_rng(seed).integers(0, T + 1, size=B).astype(np.int32)
    ln[0] = T
    w, d = _case(seed, B, T, Z, H, A, K, ln)
    _check(w, d, f"slices {B * T} rows")


@pytest.mark.parametrize("K", [1, 3, 5, 8])
def test_nll_large_tiles(K):
    w = wl.Workload("s", "nll", B=301, T=41, Z=40, H=80, A=7, K=K, dtype="fp32", seed=50 + K)
    d = wl.make_nll_inputs(w)
    m = wmlib.pack(d["weights"], w.Z, w.H, w.A, w.K, "fp32")
    t = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()  # noqa: E731
    b = wmlib.nll(m, t(d["z"]), t(d["actions"]), t(d["rewards"]), t(d["dones"]))
    torch.cuda.synchronize()
    ref = owm.nll(d["weights"], w.dims, d["z"], d["actions"], d["rewards"], d["dones"], dtype="fp32")
    for k in ("loglik", "reward_se", "done_bce", "means"):
        parity.close(getattr(b, k).cpu().numpy(), ref[k], parity.RTOL["fp32"], k)


@pytest.mark.parametrize("B,T,Z,H,A", [
    (37, 16, 40, 48, 5),    # 16-row tiles; H and Z end inside a slice of 32 columns
    (1, 16, 8, 16, 1),      # the smallest of everything
    (300, 8, 24, 272, 7),   # 16-row tiles, the last row block short
    (530, 8, 136, 528, 9),  # 32-row tiles; five slices of z
    (90, 4, 72, 1040, 2),   # weights that do not fit the L2s in eighths
    (3, 515, 40, 48, 2),    # planes of z in three rounds of steps
    (512, 9, 64, 512, 64),  # a batch that the persistent kernel also serves
])
def test_recurrence_per_step(B, T, Z, H, A):
    """The recurrence of one launch per step (with actions outside [0, A): no
    column), and the gradient of the same call."""
    w = wl.Workload("r", "nll", B=B, T=T, Z=Z, H=H, A=A, K=2, dtype="fp32", seed=60 + B)
    d = wl.make_nll_inputs(w)
    a = d["actions"].copy()
    a[0, 0], a[-1, -1] = -1, A
    d["actions"] = a
    t = lambda x: torch.from_numpy(np.ascontiguousarray(x)).cuda()  # noqa: E731
    m = wmlib.pack(d["weights"], Z, H, A, 2, "fp32")
    wmlib.profile_reset()
    wmlib.profile_enable("")
    try:
        b = wmlib.nll(m, t(d["z"]), t(a), t(d["rewards"]), t(d["dones"]))
        torch.cuda.synchronize()
        assert wmlib.profile_read("nll_step")[1] == T
    finally:
        wmlib.profile_enable(None)
        wmlib.profile_reset()
    ref = owm.nll(d["weights"], w.dims, d["z"], a, d["rewards"], d["dones"], dtype="fp32")
    for k in ("loglik", "reward_se", "done_bce", "means"):
        parity.close(getattr(b, k).cpu().numpy(), ref[k], parity.RTOL["fp32"], k)
    if T * B <= 4500:
        d["lengths"] = None
        _check(w, d, f"per-step B {B} H {H}")


@pytest.mark.parametrize("B,T,Z,H,steps", [
    (37, 15, 40, 48, 0), (37, 16, 40, 48, 16),        # few rows, small H
    (300, 7, 24, 272, 0), (300, 8, 24, 272, 8),
    (43, 3, 16, 768, 0), (43, 4, 16, 768, 4),         # large H
    (1030, 17, 8, 176, 0), (1030, 8, 8, 208, 8),      # many rows, small H
    (512, 7, 64, 512, 0),                             # the persistent kernel
])
def test_recurrence_route(B, T, Z, H, steps):
    """Few steps do not pay for splitting the operands: fp32 gate launches."""
    w = wl.Workload("q", "nll", B=B, T=T, Z=Z, H=H, A=6, K=1, dtype="fp32", seed=80 + T)
    d = wl.make_nll_inputs(w)
    t = lambda x: torch.from_numpy(np.ascontiguousarray(x)).cuda()  # noqa: E731
    m = wmlib.pack(d["weights"], Z, H, 6, 1, "fp32")
    wmlib.profile_reset()
    wmlib.profile_enable("nll_step")
    try:
        b = wmlib.nll(m, t(d["z"]), t(d["actions"]), t(d["rewards"]), t(d["dones"]))
        torch.cuda.synchronize()
        assert wmlib.profile_read("nll_step")[1] == steps
    finally:
        wmlib.profile_enable(None)
        wmlib.profile_reset()
    ref = owm.nll(d["weights"], w.dims, d["z"], d["actions"], d["rewards"], d["dones"], dtype="fp32")
    for k in ("loglik", "reward_se", "done_bce", "means"):
        parity.close(getattr(b, k).cpu().numpy(), ref[k], parity.RTOL["fp32"], k)


@pytest.mark.parametrize("B,T,Z,H,K", [
    (300, 8, 24, 272, 2),    # 16-row tiles of the recurrence
    (530, 8, 136, 528, 3),   # 32-row tiles, several slices per wave
    (512, 9, 64, 512, 5),    # a batch that the persistent kernel also serves
])
def test_infinities_as_fp32_products(B, T, Z, H, K):
    """Split products multiply infinities, and values that round to one in
    bf16, as fp32 products do: a latent saturates the gates of its row and the
    later steps stay finite; a weight moves its own logit."""
    w = wl.Workload("i", "nll", B=B, T=T, Z=Z, H=H, A=5, K=K, dtype="fp32", seed=70 + K)
    d = wl.make_nll_inputs(w)
    d["z"][0, 3, 1], d["z"][0, B - 1, Z - 1] = np.inf, -np.inf
    d["z"][1, 20, 0], d["z"][0, 33, Z // 2] = 3.4e38, -3.4e38  # above the largest bf16
    d["z"][0, 40, 2] = np.nan
    # a mixture weight whose logit (3.4e38 h) swamps the others of its dim
    d["weights"]["W_m"][0, 7] = 3.4e38
    t = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()  # noqa: E731
    m = wmlib.pack(d["weights"], Z, H, 5, K, "fp32")
    b = wmlib.nll(m, t(d["z"]), t(d["actions"]), t(d["rewards"]), t(d["dones"]))
    torch.cuda.synchronize()
    with np.errstate(all="ignore"):
        ref = owm.nll(d["weights"], w.dims, d["z"], d["actions"], d["rewards"], d["dones"], dtype="fp32")
    for k in ("loglik", "reward_se", "done_bce"):
        got, want = getattr(b, k).cpu().numpy(), ref[k]
        ok = np.isfinite(want) & (np.abs(want) < 1e30)
        assert ok[:, [3, B - 1, 33]].any() and not ok[:, 40].any(), k
        np.testing.assert_array_equal(np.isfinite(got) & (np.abs(got) < 1e30), ok, err_msg=k)
        parity.close(got[ok], want[ok], parity.RTOL["fp32"], k)
