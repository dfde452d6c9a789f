"""GPU parity of the per-step kernels on every gate and mixture tile that the
dispatch by tiles per CU can pick, each asserted by the name of its launches,
with ragged row and weight-row edges (4 H = 4032 rows: 63 tiles of 64, 31.5 of
128, 15.75 of 256), re-anchored against the oracle on a spread of rows and the
last ones."""

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


# B, Z, H, A, K, dtype, gate tile, mixture tile
TILES = [
    (15, 24, 1008, 20, 8, "bf16", "rd16", "rd"),
    (61, 24, 1008, 20, 8, "bf16", "rd32", "rd"),
    (101, 24, 1008, 20, 8, "bf16", "64x32", "rd"),
    (251, 64, 1008, 20, 8, "bf16", "64x64", "rd"),
    (499, 64, 1008, 20, 8, "bf16", "128x64", "32"),
    (701, 64, 1008, 20, 6, "bf16", "128x128", "32"),        # odd block count
    (2011, 64, 1008, 20, 8, "bf16", "128x128", "64"),
    (2011, 64, 1008, 20, 7, "bf16", "128x128", "64"),
    (2811, 128, 1008, 20, 6, "bf16", "128x128", "64"),      # odd block count
    (5003, 128, 112, 20, 8, "bf16", "128x128", "128"),
    (4001, 24, 1008, 20, 8, "bf16", "256x256/8", "64"),
    (8003, 24, 1008, 20, 5, "bf16", "256x256/16", "64"),
    (135, 128, 112, 20, 1, "fp32", "rd16", "16"),
    (301, 128, 112, 20, 3, "fp32", "rd32", "32"),
    (301, 40, 368, 20, 3, "fp32", "64x32", "rd"),
    (701, 24, 240, 20, 3, "fp32", "64x64", "16"),
    (1203, 24, 112, 20, 5, "fp32", "64x64", "32"),
    (803, 24, 1008, 20, 5, "fp32", "128x64", "16"),
    (1203, 128, 112, 20, 6, "fp32", "64x64", "128"),        # odd block count
    (4001, 40, 112, 20, 8, "fp32", "128x64", "128"),
]


@pytest.mark.parametrize("B,Z,H,A,K,dtype,gate,mix", TILES)
def test_tiles(B, Z, H, A, K, dtype, gate, mix, monkeypatch):
    print("[gpu-tiles]", B, Z, H, A, K, dtype, gate, mix, flush=True)
    sys.stdout.flush()
    monkeypatch.setenv("WM_PERSISTENT", "0")  # the per-step kernels
    w, inp = _case(B, 2, Z, H, A, K, dtype)
    m = wmlib.pack(inp["weights"], Z, H, A, K, dtype)
    cuda = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()  # noqa: E731
    rng = np.random.default_rng(B)
    h0 = np.tanh(rng.standard_normal((B, H))).astype(np.float32)
    c0 = rng.standard_normal((B, H)).astype(np.float32)
    done0 = (np.arange(B) % 7 == 3).astype(np.uint8)  # frozen rows in every tile
    wmlib.profile_reset()
    wmlib.profile_enable("")
    try:
        b = wmlib.rollout(m, cuda(inp["z0"]), cuda(inp["mask"]), T=2, seed=41, tau=1.2, done=True, trace=True,
                          h0=cuda(h0), c0=cuda(c0), done_io=cuda(done0))
        torch.cuda.synchronize()
        assert wmlib.profile_read("gates/" + gate)[1] == wmlib.profile_read("gates")[1] == 2, "gate tile"
        assert wmlib.profile_read("mdn/" + mix)[1] == wmlib.profile_read("mdn")[1] == 2, "mixture tile"
    finally:
        wmlib.profile_enable(None)
        wmlib.profile_reset()
    rows = np.unique(np.concatenate([np.linspace(0, B - 1, 40).astype(np.int64), np.arange(max(0, B - 20), B)]))
    ri = torch.from_numpy(rows).cuda()
    g = {k: getattr(b, k)[:, ri].cpu().numpy()
         for k in ("z_out", "actions", "rewards", "dones", "h_trace", "c_trace")}
    ties, live = parity.reanchored(w.dims, inp["weights"], inp["mask"][rows], g, seed=41, tau=1.2, done_flag=True,
                                   dtype=dtype, traj=rows, done0=done0[rows])
    assert live > 0


# B, Z, H, A (or N, L), K: fp32 controllers whose h part comes from the mixture
# launches
H_PART = [
    (1, 8, 64, 1, 0, 0, 1),          # one row, one action
    (33, 40, 64, 61, 0, 0, 3),       # Z ends inside a K slice; reward row in the next block
    (100, 72, 192, 62, 0, 0, 8),     # three K slices of z; A + 2 = 64
    (301, 128, 256, 300, 0, 0, 5),   # two rounds of blocks per wave
    (45, 64, 704, 766, 0, 0, 2),     # many rounds; as many logits as an activation row has columns
    (77, 24, 128, 0, 9, 30, 3),      # two levels
    (130, 64, 256, 0, 80, 200, 8),
]


@pytest.mark.parametrize("B,Z,H,A,N,L,K", H_PART)
def test_controller_h_part(B, Z, H, A, N, L, K, monkeypatch):
    """Per-step rollouts with the controller's h part beside the mixture, from
    a given state, against the oracle."""
    print("[gpu-tiles] h part", B, Z, H, A, N, L, K, flush=True)
    monkeypatch.setenv("WM_PERSISTENT", "0")
    cuda = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()  # noqa: E731
    T = 3
    if N:
        A = N * L
        w, z0, xm, lm = two_level_inputs(B, T, Z, H, N, L, K, seed=B)
        mask, dmask, dims = (xm, lm), (cuda(xm), cuda(lm)), dict(Z=Z, H=H, A=A, K=K)
        kw = dict(two_level=(N, L))
    else:
        wk, inp = _case(B, T, Z, H, A, K, "fp32")
        w, z0, mask, dims, kw = inp["weights"], inp["z0"], inp["mask"], wk.dims, {}
        dmask = cuda(mask)
    m = wmlib.pack(w, Z, H, A, K, "fp32", N=N, L=L)
    rng = np.random.default_rng(B)
    h0 = np.tanh(rng.standard_normal((B, H))).astype(np.float32)
    done0 = (np.arange(B) % 5 == 2).astype(np.uint8)
    wmlib.profile_reset()
    wmlib.profile_enable("lh")
    try:
        b = wmlib.rollout(m, cuda(z0), dmask, T=T, seed=43, tau=1.0, done=True, trace=True, h0=cuda(h0),
                          done_io=cuda(done0))
        torch.cuda.synchronize()
        assert wmlib.profile_read("lh")[1] == 1  # step 0's, from h0
    finally:
        wmlib.profile_enable(None)
        wmlib.profile_reset()
    g = {k: getattr(b, k).cpu().numpy() for k in ("z_out", "actions", "rewards", "dones", "h_trace", "c_trace")}
    parity.reanchored(dims, w, mask, g, seed=43, tau=1.0, done_flag=True, dtype="fp32", done0=done0, **kw)


@pytest.mark.parametrize("B,Z,H,A,h0", [
    (300, 128, 1024, 400, True),
    (1300, 128, 4096, 1030, False),  # 65 MB of workspace: what the static scratch just holds
])
def test_controller_sums_do_not_follow_the_workspace(B, Z, H, A, h0):
    """The controller's h part waits in the activation buffers: a call on the
    static scratch, or in a larger workspace, has the same bits, and wm_rollout
    refuses a workspace below wm_workspace_bytes."""
    print("[gpu-tiles] workspace", B, Z, H, A, h0, flush=True)
    g = torch.Generator(device="cuda").manual_seed(B)
    shapes = dict(W_g=(4 * H, Z + A + H), b_g=(4 * H,), W_m=(6 * Z, H), b_m=(6 * Z,), w_r=(H,), b_r=(1,), w_d=(H,),
                  b_d=(1,), W_c=(A, Z + H), b_c=(A,))
    w = {k: torch.randn(s, generator=g, device="cuda") / H ** 0.5 for k, s in shapes.items()}
    m = wmlib.pack(w, Z, H, A, 2, "fp32")
    z0 = torch.randn((B, Z), generator=g, device="cuda")
    mask = torch.ones((B, A), dtype=torch.uint8, device="cuda")
    kw = dict(T=2, seed=3, done=False, h0=torch.tanh(torch.randn((B, H), generator=g, device="cuda")) if h0 else None)
    need = wmlib.workspace_bytes(m.dims, B, 2, wmlib.WS_ROLLOUT)
    assert need <= 64 << 20
    big = wmlib.RolloutBuffers(m, B, 2)
    assert big.ws_bytes == need
    big.workspace, big.ws_bytes = torch.empty(need + (16 << 20), dtype=torch.uint8, device="cuda"), need + (16 << 20)
    out = [wmlib.rollout(m, z0, mask, **kw), wmlib.rollout(m, z0, mask, bufs=big, **kw),
           wmlib.rollout(m, z0, mask, noalloc=True, **kw)]
    torch.cuda.synchronize()
    for o in out[1:]:
        for k in ("actions", "rewards", "z_out", "h_T", "c_T"):
            assert torch.equal(getattr(o, k), getattr(out[0], k)), k
    big.ws_bytes = need - 1
    with pytest.raises(wmlib.WmError) as e:
        wmlib.rollout(m, z0, mask, bufs=big, **kw)
    assert e.value.status == wmlib.WM_ERR_WORKSPACE
