"""What a bf16 call's results do not depend on: the tile that its size runs
on.  The order of the sums and the LSTM cell's arithmetic follow the class of
its rows (at most 256, more), so that one trajectory gives the same bits in
batches of one class whichever kernel serves them, a NaN stays a NaN, and c,
which is fp32 state, keeps the accuracy of the separate sigmoids and tanhs."""

import sys

import numpy as np
import pytest
import torch

from paper_2205_01435_amd import _lib as wmlib
from test_gpu_edges import _case

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def gpu():
    assert torch.cuda.is_available(), "GPU tests need a ROCm GPU"
    wmlib.load()
    yield


def _cuda(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def _state(B, H, seed):
    rng = np.random.default_rng(seed)
    return (np.tanh(rng.standard_normal((B, H))).astype(np.float32),
            rng.standard_normal((B, H)).astype(np.float32))


# B (the larger batch), b (the smaller one), Z, H
GATES = [
    (256, 33, 64, 1024),  # 64 x 64 tiles against register-direct ones; runs of four slices
    (250, 64, 24, 512),   # ragged rows; the last wave's run is empty
    (100, 31, 8, 1040),   # 64 x 32 tiles, a ragged unit block
    (256, 16, 40, 1216),  # 128 x 64 tiles
    (256, 20, 64, 448),   # runs of two slices
]


@pytest.mark.parametrize("B,b,Z,H", GATES)
def test_gate_sums_do_not_follow_the_tile(B, b, Z, H):
    print("[gpu-rounding] gates", B, b, Z, H, flush=True)
    sys.stdout.flush()
    w, inp = _case(B, 1, Z, H, 20, 3, "bf16")
    m = wmlib.pack(inp["weights"], Z, H, 20, 3, "bf16")
    h0, c0 = _state(B, H, B)
    done = (np.arange(B) % 7 == 3).astype(np.uint8)
    out = []
    for n in (B, b):
        r = wmlib.rollout(m, _cuda(inp["z0"][:n]), _cuda(inp["mask"][:n]), T=1, seed=7, h0=_cuda(h0[:n]),
                          c0=_cuda(c0[:n]), done_io=_cuda(done[:n]))
        torch.cuda.synchronize()
        out.append((r.actions[0, :b], r.h_T[:b], r.c_T[:b]))
    for x, y in zip(*out):
        assert torch.equal(x, y)


@pytest.mark.parametrize("B,H", [(48, 1024), (200, 1024), (256, 512)])
def test_nan_latent_reaches_the_state(B, H):
    """A NaN in a row's latent makes its h and c NaN, and no other row's."""
    print("[gpu-rounding] nan", B, H, flush=True)
    w, inp = _case(B, 1, 16, H, 20, 2, "bf16")
    m = wmlib.pack(inp["weights"], 16, H, 20, 2, "bf16")
    acts = np.zeros((1, B), np.int32)
    z = np.random.default_rng(B).standard_normal((2, B, 16)).astype(np.float32)
    z[0, B - 2, 5] = np.nan
    # the likelihood pass takes the actions as given, so that the row steps on
    o = wmlib.nll(m, _cuda(z), _cuda(acts), _cuda(np.zeros((1, B), np.float32)), _cuda(np.zeros((1, B), np.uint8)))
    torch.cuda.synchronize()
    bad = np.arange(B) == B - 2
    np.testing.assert_array_equal(np.isnan(o.reward_se[0].cpu().numpy()), bad)
    np.testing.assert_array_equal(np.isnan(o.loglik[0].cpu().numpy()), bad)


def test_saturated_gates_keep_c():
    """c' = sigmoid(f) c + sigmoid(i) tanh(g) from pre-activations out to +-25,
    exact in the biases (no product): each factor is within 1e-6 of its size
    (fsigmoid) or 5e-7 (ftanh_abs), where a cell that clamps at +-15 is off by
    3e-7 of c itself."""
    B, Z, H = 256, 16, 1024
    w, inp = _case(B, 1, Z, H, 4, 1, "bf16")
    wt = {k: np.zeros_like(v) for k, v in inp["weights"].items()}
    rng = np.random.default_rng(3)
    bg = rng.uniform(-25, 25, 4 * H).astype(np.float32)
    wt["b_g"] = bg
    m = wmlib.pack(wt, Z, H, 4, 1, "bf16")
    h0, c0 = _state(B, H, 5)
    r = wmlib.rollout(m, _cuda(inp["z0"]), _cuda(np.ones((B, 4), np.uint8)), T=1, seed=1, h0=_cuda(h0), c0=_cuda(c0))
    torch.cuda.synchronize()
    i, f, g, _ = np.split(bg.astype(np.float64), 4)
    sig = lambda x: 1.0 / (1.0 + np.exp(-x))  # noqa: E731
    a, b = sig(f) * c0.astype(np.float64), sig(i) * np.tanh(g)
    err = np.abs(r.c_T.cpu().numpy() - (a + b))
    # 2^-23: the rounding of the sum
    bound = 1e-6 * np.abs(a) + sig(i) * (1e-6 * np.abs(np.tanh(g)) + 5e-7) + 2.0 ** -23 * np.abs(a + b) + 1e-30
    assert np.all(err <= bound), float((err / bound).max())


# B, b, Z, H, A, K: the controller on staged tiles, on register-direct ones
CTRL = [(256, 48, 64, 1024, 128, 8), (250, 40, 32, 512, 24, 4), (130, 16, 24, 1024, 200, 3)]


@pytest.mark.parametrize("B,b,Z,H,A,K", CTRL)
def test_rewards_do_not_follow_the_batch(B, b, Z, H, A, K):
    """The reward logits are rows of the controller's product: the bits of a
    transition's reward are those of its own row."""
    print("[gpu-rounding] rewards", B, b, Z, H, A, K, flush=True)
    w, inp = _case(B, 2, Z, H, A, K, "bf16")
    m = wmlib.pack(inp["weights"], Z, H, A, K, "bf16")
    h0 = _state(B, H, B)[0]
    out = []
    for n in (B, b):
        r = wmlib.rollout(m, _cuda(inp["z0"][:n]), _cuda(inp["mask"][:n]), T=2, seed=7, done=False,
                          h0=_cuda(h0[:n]))
        torch.cuda.synchronize()
        out.append((r.actions[:, :b], r.rewards[:, :b], r.z_out[:, :b]))
    for x, y in zip(*out):
        assert torch.equal(x, y)


# B (64- or 32-row tiles), b (register-direct up to 1024 rows, else 32-row
# tiles), Z, H, K; h of 257 rows and more comes from the same chain of sums
MIX = [
    (1000, 300, 64, 512, 8),    # runs of four slices
    (1024, 257, 40, 1008, 7),   # an odd block count, ragged rows
    (600, 260, 128, 80, 3),     # runs of one slice, the last wave's empty
    (2048, 1030, 64, 512, 8),   # even and odd slices
    (1500, 1100, 16, 1344, 5),  # K too deep for the register-direct tiles
    (900, 300, 72, 1344, 2),
]


@pytest.mark.parametrize("B,b,Z,H,K", MIX)
def test_mixture_sums_do_not_follow_the_tile(B, b, Z, H, K):
    print("[gpu-rounding] mixture", B, b, Z, H, K, flush=True)
    w, inp = _case(B, 1, Z, H, 20, K, "bf16")
    m = wmlib.pack(inp["weights"], Z, H, 20, K, "bf16")
    h0, c0 = _state(B, H, B)
    out = []
    for n in (B, b):
        r = wmlib.rollout(m, _cuda(inp["z0"][:n]), _cuda(inp["mask"][:n]), T=1, seed=7, done=False, h0=_cuda(h0[:n]),
                          c0=_cuda(c0[:n]))
        torch.cuda.synchronize()
        out.append((r.actions[0, :b], r.h_T[:b], r.z_out[1, :b]))
    for x, y in zip(*out):
        assert torch.equal(x, y)
