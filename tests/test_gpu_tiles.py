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
