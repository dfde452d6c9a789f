"""GPU parity of the per-step kernels on every gate and mixture tile: one call
per tile that the dispatch by tiles per CU can pick, with ragged row and
weight-row edges (4 H = 4032 rows: 63 tiles of 64, 31.5 of 128, 15.75 of 256),
re-anchored against the oracle on a spread of rows and the last ones."""

import sys

import numpy as np
import pytest
import torch

import parity
from paper_2205_01435_amd import _lib as wmlib
from test_gpu_edges import _case
from test_gpu_two_level import _inputs as two_level_inputs

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def gpu():
    assert torch.cuda.is_available(), "GPU tests need a ROCm GPU"
    wmlib.load()
    yield


# B, Z, H, A, K, dtype   (gate tile / mixture tile)
TILES = [
    (15, 24, 1008, 20, 8, "bf16"),     # register-direct 16 / register-direct
    (61, 24, 1008, 20, 8, "bf16"),     # register-direct 32 / register-direct
    (101, 24, 1008, 20, 8, "bf16"),    # 64 x 32 / register-direct
    (251, 64, 1008, 20, 8, "bf16"),    # 64 x 64 / register-direct
    (499, 64, 1008, 20, 8, "bf16"),    # 128 x 64 / 32 rows
    (701, 64, 1008, 20, 6, "bf16"),    # 128 x 128 / 32 rows, odd block count
    (2011, 64, 1008, 20, 8, "bf16"),   # 128 x 128 / 64 rows
    (2011, 64, 1008, 20, 7, "bf16"),   # the same, K 7
    (2811, 128, 1008, 20, 8, "bf16"),  # 128 x 128 / 128 rows
    (2811, 128, 1008, 20, 6, "bf16"),  # 128 x 128 / 64 rows, odd block count
    (4001, 24, 1008, 20, 8, "bf16"),   # 256 x 256, eight waves / 64 rows
    (8003, 24, 1008, 20, 5, "bf16"),   # 256 x 256, sixteen waves / 128 rows
    (301, 40, 368, 20, 3, "fp32"),     # 64 x 32 / register-direct beyond one per CU: 16 rows
    (500, 64, 528, 20, 5, "fp32"),     # 64 x 64 / 16 rows
    (2003, 24, 528, 20, 5, "fp32"),    # 128 x 64 / 32 rows
]


@pytest.mark.parametrize("B,Z,H,A,K,dtype", TILES)
def test_tiles(B, Z, H, A, K, dtype, monkeypatch):
    print("[gpu-tiles]", B, Z, H, A, K, dtype, flush=True)
    sys.stdout.flush()
    monkeypatch.setenv("WM_PERSISTENT", "0")  # the per-step kernels
    w, inp = _case(B, 2, Z, H, A, K, dtype)
    m = wmlib.pack(inp["weights"], Z, H, A, K, dtype)
    cuda = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()  # noqa: E731
    rng = np.random.default_rng(B)
    h0 = np.tanh(rng.standard_normal((B, H))).astype(np.float32)
    c0 = rng.standard_normal((B, H)).astype(np.float32)
    done0 = (np.arange(B) % 7 == 3).astype(np.uint8)  # frozen rows in every tile
    b = wmlib.rollout(m, cuda(inp["z0"]), cuda(inp["mask"]), T=2, seed=41, tau=1.2, done=True, trace=True,
                      h0=cuda(h0), c0=cuda(c0), done_io=cuda(done0))
    torch.cuda.synchronize()
    rows = np.unique(np.concatenate([np.linspace(0, B - 1, 40).astype(np.int64), np.arange(max(0, B - 20), B)]))
    ri = torch.from_numpy(rows).cuda()
    g = {k: getattr(b, k)[:, ri].cpu().numpy()
         for k in ("z_out", "actions", "rewards", "dones", "h_trace", "c_trace")}
    ties, live = parity.reanchored(w.dims, inp["weights"], inp["mask"][rows], g, seed=41, tau=1.2, done_flag=True,
                                   dtype=dtype, traj=rows, done0=done0[rows])
    assert live > 0


# B, Z, H, A (or N, L), K, dtype: controllers whose h part comes from the
# mixture launches
H_PART = [
    (1, 8, 64, 1, 0, 0, 1, "fp32"),          # one row, one action
    (33, 40, 64, 61, 0, 0, 3, "fp32"),       # Z ends inside a K slice; reward row in the next block
    (100, 72, 192, 62, 0, 0, 8, "fp32"),     # three K slices of z; A + 2 = 64
    (301, 128, 256, 300, 0, 0, 5, "fp32"),   # two rounds of blocks per wave
    (45, 16, 64, 1500, 0, 0, 2, "fp32"),     # many rounds
    (77, 24, 128, 0, 9, 30, 3, "fp32"),      # two levels
    (130, 64, 256, 0, 80, 200, 8, "fp32"),
]


@pytest.mark.parametrize("B,Z,H,A,N,L,K,dtype", H_PART)
def test_controller_h_part(B, Z, H, A, N, L, K, dtype, monkeypatch):
    """Per-step rollouts with the controller's h part beside the mixture, from
    a given state, against the oracle, and against the same call in a
    workspace that has no room for it."""
    print("[gpu-tiles] h part", B, Z, H, A, N, L, K, dtype, flush=True)
    monkeypatch.setenv("WM_PERSISTENT", "0")
    cuda = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()  # noqa: E731
    T = 3
    if N:
        A = N * L
        w, z0, xm, lm = two_level_inputs(B, T, Z, H, N, L, K, seed=B)
        mask, dmask, dims = (xm, lm), (cuda(xm), cuda(lm)), dict(Z=Z, H=H, A=A, K=K)
        kw = dict(two_level=(N, L))
    else:
        wk, inp = _case(B, T, Z, H, A, K, dtype)
        w, z0, mask, dims, kw = inp["weights"], inp["z0"], inp["mask"], wk.dims, {}
        dmask = cuda(mask)
    m = wmlib.pack(w, Z, H, A, K, dtype, N=N, L=L)
    rng = np.random.default_rng(B)
    h0 = np.tanh(rng.standard_normal((B, H))).astype(np.float32)
    done0 = (np.arange(B) % 5 == 2).astype(np.uint8)
    args = dict(T=T, seed=43, tau=1.0, done=True, trace=True, h0=cuda(h0))
    out = []
    ac = N + 1 + L if N else A
    part = (B * ((ac + 2 + 15) // 16 * 16) * 4 + 255) // 256 * 256
    for less in (0, part):
        b = wmlib.RolloutBuffers(m, B, T, trace=True)
        b.ws_bytes -= less
        wmlib.rollout(m, cuda(z0), dmask, bufs=b, done_io=cuda(done0), **args)
        torch.cuda.synchronize()
        out.append({k: getattr(b, k).cpu().numpy()
                    for k in ("z_out", "actions", "rewards", "dones", "h_trace", "c_trace")})
        parity.reanchored(dims, w, mask, out[-1], seed=43, tau=1.0, done_flag=True, dtype=dtype, done0=done0, **kw)
    same = np.all(out[0]["actions"] == out[1]["actions"], axis=0)
    assert same.mean() >= 0.97
