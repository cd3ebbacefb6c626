"""Global selection spread over the chip (more than 32768 blocks): histogram window, candidate
list and placement, bit for bit against the oracle.

The kinds aim at the places where the selection changes course: a threshold inside the window,
below it (an outlier or widely spread magnitudes push most keys into the first bin), above it
(infinities and NaN), more equal keys than are ranked directly, a bin with more distinct keys
than the candidate list holds, and zero blocks kept because k exceeds the nonzero ones.
"""
import numpy as np
import pytest

from paper_2106_08846_amd import bsr as B

from .gpu_common import check_prune, dev, host, log, O

pytestmark = pytest.mark.gpu


def weights(kind: str, N: int, K: int) -> np.ndarray:
    g = np.random.Generator(np.random.PCG64(N + K + len(kind)))
    W = (g.standard_normal((N, K)) * 0.02).astype(np.float32)
    if kind == "ties":
        W = g.integers(-2, 3, (N, K)).astype(np.float32)
    elif kind == "zeros":
        W[g.random((N, K)) < 0.7] = 0.0
    elif kind == "narrow":    # keys in [1, 1 + 2^-15): one bin of any octave-wide window
        W = (1.0 + g.random((N, K)) * 2.0 ** -16).astype(np.float32)
        W[0, 0] = 1e12        # the window starts far above them
    elif kind == "spread":
        W = (W * np.exp2(g.integers(-60, 60, (N, K)))).astype(np.float32)
    elif kind == "nonfinite":
        flat = W.reshape(-1)
        idx = g.choice(flat.size, 12, replace=False)
        flat[idx[:4]], flat[idx[4:8]], flat[idx[8:]] = np.nan, np.inf, -np.inf
    return W


SHAPES = [(3, 10923, 1, 1),      # 32769 blocks: the smallest of the range
          (1030, 1031, 1, 1),    # ragged chunks
          (1152, 768, 4, 4),     # 55296 blocks of 16 elements
          (2112, 1024, 32, 1)]   # 67584 tall blocks


@pytest.mark.parametrize("shape", SHAPES, ids=[f"{s[0]}x{s[1]}_{s[2]}x{s[3]}" for s in SHAPES])
@pytest.mark.parametrize("kind", ["normal", "ties", "zeros", "narrow", "spread", "nonfinite"])
def test_wide_select_bit_exact(device, shape, kind):
    N, K, R, C = shape
    nb = (N // R) * (K // C)
    W = weights(kind, N, K)
    Wd = dev(W)
    for k in sorted({1, 5, nb // 10, nb // 2, nb - 1, nb}):
        log(f"wide select {kind} {N}x{K} {R}x{C} nb={nb} k={k}")
        check_prune(W, R, C, B.bsr_prune_from_dense(Wd, R, C, k=k), k)


def test_wide_select_l1_pitched_unaligned(device):
    """l1 keys, a pitched W, and a workspace that starts at an odd address."""
    N, K, R, C = 520, 300, 2, 2
    big = np.random.Generator(np.random.PCG64(5)).standard_normal((N, K + 7)).astype(np.float32)
    W = np.ascontiguousarray(big[:, :K])
    k = 9001
    ws = B.torch.empty(B.bsr_prune_workspace_bytes(N, K, R, C) + 8, dtype=B.torch.uint8,
                       device="cuda:0")
    log("wide select l1, pitched W, workspace at + 8 bytes")
    M = B.bsr_prune_from_dense(dev(big)[:, :K], R, C, k=k, norm="l1", workspace=ws[8:])
    ids = O.select_topk(O.block_keys(W, R, C, norm="l1"), k)
    ip, ix, dt = O.build_bsr(W, R, C, ids)
    assert np.array_equal(host(M.indptr), ip)
    assert np.array_equal(host(M.indices)[:k], ix)
    assert np.array_equal(host(M.data)[:k].view(np.uint32), dt.view(np.uint32))


def test_wide_select_large(device):
    """2.4 million one-element blocks: chunk counts and the candidate list at a real size."""
    W = weights("normal", 3072, 768)
    log("wide select 3072x768 1x1")
    check_prune(W, 1, 1, B.bsr_prune_from_dense(dev(W), 1, 1, k=235930), 235930)
