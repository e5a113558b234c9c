"""GPU parity: dass_down_proj_sparse24 (Eq. 3 from the 2:4 compressed Down-Proj on the sparse
matrix cores) against the float64 oracle.

Tolerance, derived from the arithmetic (u = 2^-8, bf16's unit roundoff; A = the sum of the
magnitudes of the terms, from the oracle): the products are exact in f32, their f32 accumulation
errs by at most K 2^-24 A <= 0.44 u A for K = d_int <= 28672 (worst-case linear bound), and the
output is rounded to bf16 once: |gpu - oracle| <= u |oracle| + 0.5 u A.
"""
import numpy as np
import pytest
import torch

import oracle
import paper_2405_01943_amd as dass
from paper_2405_01943_amd import synth

from gpu_helpers import padded, to_np32

pytestmark = pytest.mark.gpu


def _check(out, ref, ab, what):
    tol = 2.0 ** -8 * (np.abs(ref) + 0.5 * ab) + 1e-30
    err = np.abs(np.asarray(out, dtype=np.float64) - ref)
    worst = float(np.max(err / tol))
    assert worst <= 1.0, f"{what}: worst error / tolerance = {worst:.3f}"
    assert float(np.mean(err / tol)) < 0.35, what


def _sparse_weights(d, d_int, seed):
    rng = np.random.default_rng(seed)
    W = (rng.standard_normal((d, d_int)) * 0.1).astype(np.float32)
    for row in W:
        for g in range(d_int // 4):
            row[4 * g + rng.choice(4, size=2, replace=False)] = 0.0
    W[rng.random(W.shape) < 0.05] = 0.0
    return torch.from_numpy(W).to(torch.bfloat16)


# T, d, d_int, padding and the kernel's tile: 0 the largest, 1 half as many tokens, 2 half of both
SHAPES = [(300, 192, 320, 0, 2), (513, 264, 448, 8, 2), (256, 256, 64, 0, 2), (70, 8, 704, 16, 2), (1, 520, 128, 0, 2),
          (8200, 520, 192, 8, 1), (4225, 1032, 576, 0, 1), (33100, 512, 128, 0, 0)]
TILE_SHAPES = [(T, d, tile) for T, d, _, _, tile in SHAPES]


@pytest.mark.parametrize("T,d,d_int,pad", [shape[:4] for shape in SHAPES])
def test_sparse_down_small_shapes(gpu_device, T, d, d_int, pad):
    W = _sparse_weights(d, d_int, T + d)
    # the compressed form comes from the oracle, so the test does not lean on the GPU's compressor
    ov, om, surplus = oracle.compress_24(W.float().numpy(), "cols")
    assert surplus == 0
    values = torch.from_numpy(ov).to(torch.bfloat16).to(gpu_device)
    meta = torch.from_numpy(om).to(gpu_device)
    g = torch.Generator(device="cpu").manual_seed(d_int)
    Y = torch.randn((T, d_int), generator=g).to(torch.bfloat16).to(gpu_device)
    out = torch.full((T, d), 3.0, dtype=torch.bfloat16, device=gpu_device)
    if pad:
        Y, values, out = padded(Y, pad), padded(values, pad), padded(out, pad)
        big = torch.full((d, d_int // 8 + 4), 0xEE, dtype=torch.uint8, device=gpu_device)
        big[:, :d_int // 8] = meta
        meta = big[:, :d_int // 8]
    dass.down_proj_sparse24(Y, values, meta, out)
    torch.cuda.synchronize()
    ref, ab = oracle.down_sparse24(to_np32(Y), ov, om, want_abs=True)
    _check(to_np32(out), ref, ab, f"T={T} d={d} d_int={d_int}")
    if pad:
        assert torch.all(out._base[:, d:] == 7.0)


@pytest.mark.parametrize("T,d", [(90, 136), (8200, 520), (33100, 512)])
@pytest.mark.parametrize("slabs", [1, 2, 3, 4, 5, 6, 7, 8, 9, 10, 11, 12, 13, 14, 15, 16, 17])
@pytest.mark.parametrize("pad", [0, 8])
def test_sparse_down_code_blocks(gpu_device, T, d, slabs, pad):
    """K around the ends of the blocks that the position codes come in (4 and 8 slabs of 64) and of the loops that are
    unrolled by 2 and 4 slabs, all three tiles; rows longer than K too (the last unit of an odd number of slabs then
    reaches into what lies between two rows)."""
    d_int = 64 * slabs
    W = _sparse_weights(d, d_int, slabs)
    ov, om, _ = oracle.compress_24(W.float().numpy(), "cols")
    values, meta = torch.from_numpy(ov).to(torch.bfloat16).to(gpu_device), torch.from_numpy(om).to(gpu_device)
    Y = torch.randn((T, d_int), generator=torch.Generator(device="cpu").manual_seed(d_int)).to(torch.bfloat16).to(gpu_device)
    out = torch.empty((T, d), dtype=torch.bfloat16, device=gpu_device)
    if pad:
        Y, values, out = padded(Y, pad), padded(values, pad), padded(out, pad)
        meta = torch.nn.functional.pad(meta, (0, 4), value=0xEE)[:, :d_int // 8]
    dass.down_proj_sparse24(Y, values, meta, out)
    torch.cuda.synchronize()
    ref, ab = oracle.down_sparse24(to_np32(Y[-80:]), ov, om, want_abs=True)
    _check(to_np32(out[-80:]), ref, ab, f"T={T} d={d} d_int={d_int} pad={pad}")
    assert not pad or torch.all(out._base[:, d:] == 7.0)


def test_sparse_down_equals_dense_route(gpu_device):
    """Prune, compress and multiply on the GPU, and compare with the dense down projection of
    dass_mlp_forward's second launch on the same pruned matrix: the same sums in another order."""
    T, d, d_int = 700, 256, 512
    g = torch.Generator(device="cpu").manual_seed(4)
    X = torch.randn((T, d), generator=g).to(torch.bfloat16).to(gpu_device)
    Wg, Wu = ((torch.randn((d_int, d), generator=g) * 0.1).to(torch.bfloat16).to(gpu_device) for _ in range(2))
    Wd = (torch.randn((d, d_int), generator=g) * 0.1).to(torch.bfloat16).to(gpu_device)
    norms = torch.rand(d_int, generator=g).to(gpu_device) + 0.5
    dass.score_mask_nm(Wd, norms, "cols", "cols", 1.0, 2, 4)
    values = torch.empty((d, d_int // 2), dtype=torch.bfloat16, device=gpu_device)
    meta = torch.empty((d, d_int // 8), dtype=torch.uint8, device=gpu_device)
    dass.compress_24(Wd, "cols", values, meta)
    dense = torch.empty((T, d), dtype=torch.bfloat16, device=gpu_device)
    ws = torch.empty(dass.mlp_forward_workspace_bytes(T, d, d_int), dtype=torch.uint8, device=gpu_device)
    dass.mlp_forward(X, Wg, Wu, Wd, "silu", dense, workspace=ws)
    Y = ws.view(torch.bfloat16).view(T, d_int)          # the y that the dense route multiplied
    sparse = torch.empty_like(dense)
    dass.down_proj_sparse24(Y, values, meta, sparse)
    torch.cuda.synchronize()
    ref, ab = oracle.down_sparse24(to_np32(Y), to_np32(values), meta.cpu().numpy(), want_abs=True)
    _check(to_np32(sparse), ref, ab, "sparse route")
    _check(to_np32(dense), ref, ab, "dense route")


def test_eq2_only_then_sparse_down(gpu_device):
    """dass_mlp_forward without a Down-Proj stops after Eq. 2: the y it leaves in the workspace is
    bit for bit the y of the full call, and the sparse down projection of it meets the oracle's
    whole pruned block (bf16 y in between on both sides)."""
    T, d, d_int = 450, 192, 384
    g = torch.Generator(device="cpu").manual_seed(21)
    X = torch.randn((T, d), generator=g).to(torch.bfloat16).to(gpu_device)
    Wg, Wu = ((torch.randn((d_int, d), generator=g) * 0.1).to(torch.bfloat16).to(gpu_device) for _ in range(2))
    Wd = (torch.randn((d, d_int), generator=g) * 0.1).to(torch.bfloat16).to(gpu_device)
    norms = torch.rand(d_int, generator=g).to(gpu_device) + 0.5
    dass.score_mask_nm(Wd, norms, "cols", "cols", 1.0, 2, 4)
    values = torch.empty((d, d_int // 2), dtype=torch.bfloat16, device=gpu_device)
    meta = torch.empty((d, d_int // 8), dtype=torch.uint8, device=gpu_device)
    dass.compress_24(Wd, "cols", values, meta)
    nbytes = dass.mlp_forward_workspace_bytes(T, d, d_int)
    ws_full = torch.zeros(nbytes, dtype=torch.uint8, device=gpu_device)
    ws_eq2 = torch.full((nbytes,), 0x55, dtype=torch.uint8, device=gpu_device)
    dense = torch.empty((T, d), dtype=torch.bfloat16, device=gpu_device)
    dass.mlp_forward(X, Wg, Wu, Wd, "gelu_tanh", dense, workspace=ws_full)
    dass.mlp_forward(X, Wg, Wu, None, "gelu_tanh", None, workspace=ws_eq2)
    torch.cuda.synchronize()
    assert torch.equal(ws_full, ws_eq2)
    sparse = torch.empty_like(dense)
    dass.down_proj_sparse24(ws_eq2.view(torch.bfloat16).view(T, d_int), values, meta, sparse)
    torch.cuda.synchronize()
    ref, ab = oracle.mlp_forward(to_np32(X), to_np32(Wg), to_np32(Wu), to_np32(Wd), "gelu_tanh", want_abs=True)
    err = np.abs(to_np32(sparse).astype(np.float64) - ref) / (2.0 ** -8 * (np.abs(ref) + 1.05 * ab) + 1e-30)
    assert float(err.max()) <= 1.0, f"sparse block output at {err.max():.2f} of its tolerance"
    with pytest.raises(ValueError):
        dass.mlp_forward(X, Wg, Wu, None, "gelu_tanh", None)


def test_sparse_down_full_size(gpu_device):
    """LLaMA2-7B-shaped Down-Proj with DaSS 2:4 weights, 32768 tokens, sampled tokens against the
    oracle (first, last, both sides of tile boundaries, seeded random ones)."""
    cfg = synth.CONFIGS["llama2_7b"]
    dev = gpu_device
    T, d, d_int = 32768, cfg.d, cfg.d_int
    Wd = synth.make_weight(cfg, "wd", dev)
    norms = synth.make_norms(d_int, dev)
    dass.score_mask_nm(Wd, norms, "cols", "cols", 1.0, 2, 4)
    values = torch.empty((d, d_int // 2), dtype=Wd.dtype, device=dev)
    meta = torch.empty((d, d_int // 8), dtype=torch.uint8, device=dev)
    surplus = torch.zeros(1, dtype=torch.int64, device=dev)
    dass.compress_24(Wd, "cols", values, meta, surplus)
    g = torch.Generator(device=dev).manual_seed(1)
    Y = torch.randn((T, d_int), generator=g, device=dev, dtype=torch.float32).to(torch.bfloat16)
    out = torch.empty((T, d), dtype=torch.bfloat16, device=dev)
    dass.down_proj_sparse24(Y, values, meta, out)
    torch.cuda.synchronize()
    assert int(surplus.item()) == 0
    rng = np.random.default_rng(0)
    tokens = np.unique(np.concatenate([[0, 1, 255, 256, 257, 1023, 1024, T - 257, T - 256, T - 1],
                                       rng.integers(0, T, size=14)]))
    sel = torch.as_tensor(tokens, device=dev)
    ref, ab = oracle.down_sparse24(to_np32(Y[sel]), to_np32(values), meta.cpu().numpy(), want_abs=True)
    _check(to_np32(out[sel]), ref, ab, "7B shape")
    assert torch.isfinite(out.float()).all()
