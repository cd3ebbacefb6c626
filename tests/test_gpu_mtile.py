"""The matrix-core kernel for blocks of 4 or 8 rows (4x1, 8x1, 4x4, 8x8) against the oracle.

Sizes sit where it changes course (every product above the work at which the library takes it, which
the tests assert): token tiles of 32 and 64 with tails, one block-row, rows without blocks and full rows next to
each other (units cut by wave boundaries), many rows per wave, inputs wide enough for several
column chunks, layers too wide for staged stores, forced slice counts, and calls whose products
share a launch or are split over two.  Integer-valued inputs are exact in any order and must equal
the generic kernel bit for bit; an infinite X element in a column no block reads must not show.
"""
import numpy as np
import pytest
import torch

from paper_2106_08846_amd import bsr as B

from .gpu_common import check_spmm, dev, host, log

pytestmark = pytest.mark.gpu

SHAPES = [(8, 8), (4, 4), (8, 1), (4, 1)]


def matrix(N, K, R, C, density, seed, skew, integer=False):
    """Dense W with a chosen block pattern (skew: empty, sparse and full rows in turn) as BSR."""
    g = np.random.Generator(np.random.PCG64(seed))
    Nb, Kb = N // R, K // C
    mask = g.random((Nb, Kb)) < density
    if skew:
        mask[0::4] = False
        mask[1::4] = True
    W = g.integers(1, 5, (N, K)) if integer else g.standard_normal((N, K)) * 0.02 + 1e-3
    W = (W * np.kron(mask, np.ones((R, C)))).astype(np.float32)
    return B.bsr_prune_from_dense(dev(W), R, C, k=int(mask.sum()))


def inputs(T, K, seed, bf16, integer=False):
    g = np.random.Generator(np.random.PCG64(seed + 1))
    X = (g.integers(-4, 5, (T, K)) if integer else g.standard_normal((T, K))).astype(np.float32)
    Xd = dev(X)
    return X, B.bsr_cast_f32_bf16(Xd) if bf16 else Xd


CASES = [
    # T, N, K (in blocks of 8), density, skew, slices
    (24003, 8, 768, 1.0, False, None),  # one 8x8 block-row, the last tile nearly empty
    (321, 1032, 768, 0.7, False, None), # a last tile of one token
    (200, 2064, 768, 0.5, True, 1),     # one slice: rows cut between waves
    (640, 3072, 136, 0.7, True, 1),     # many rows per wave
    (129, 1032, 3072, 0.8, True, None), # several column chunks, few rows per slice
    (450, 768, 1544, 0.5, True, 2),     # chunks, rows cut by waves in every chunk
    (95, 2312, 768, 0.9, False, 72),    # four block-rows of 8 per slice
    (300, 1024, 1024, 0.5, True, 3),    # a tile that leaves no room for staged stores
]


def assert_enough_work(M, T, bf16):
    """The product is above the least work of this kernel (below it, another kernel would pass the
    test): 16 Mi multiply-adds in bf16; 128 Mi in fp32, 192 Mi where the X tile of 32 tokens does not
    fit in LDS (160 KB) and is cut into column chunks."""
    least = 16 if bf16 else 192 if 32 * 4 * M.n_cols > 150 * 1024 else 128
    assert M.nnzb * M.R * M.C * T >= least << 20, "too little work for the kernel under test"


@pytest.mark.parametrize("bf16", [False, True], ids=["f32", "bf16"])
@pytest.mark.parametrize("R,C", SHAPES, ids=[f"{r}x{c}" for r, c in SHAPES])
@pytest.mark.parametrize("case", range(len(CASES)))
def test_mtile_against_oracle(device, case, R, C, bf16):
    T, N, K, d, skew, slices = CASES[case]
    log(f"mtile {R}x{C} {'bf16' if bf16 else 'f32'} T={T} {N}x{K} d={d} skew={skew} S={slices}")
    M = matrix(N, K, R, C, d, case, skew)
    assert_enough_work(M, T, bf16)
    bias = np.linspace(-1, 1, N).astype(np.float32)
    X, Xd = inputs(T, K, case, bf16)
    if bf16:
        M = M.to_bf16()
    Y = B.bsr_spmm_ex(Xd, M, dev(bias), None, kernel=None if slices is None else 0, slices=slices)
    check_spmm(X, M, bias, Y, bf16=bf16)
    again = B.bsr_spmm_ex(Xd, M, dev(bias), None, kernel=None if slices is None else 0,
                          slices=slices)
    assert torch.equal(Y, again), "not reproducible"
    M = matrix(N, K, R, C, d, case, skew, integer=True)
    X, Xd = inputs(T, K, case, bf16, integer=True)
    if bf16:
        M = M.to_bf16()
    Yi = B.bsr_spmm_ex(Xd, M, None, None, kernel=None if slices is None else 0, slices=slices)
    assert torch.equal(Yi, B.bsr_spmm_ex(Xd, M, None, None, kernel=B.KERNEL_GENERIC))


@pytest.mark.parametrize("bf16", [False, True], ids=["f32", "bf16"])
@pytest.mark.parametrize("R,C", SHAPES, ids=[f"{r}x{c}" for r, c in SHAPES])
def test_mtile_infinities_and_pitch(device, R, C, bf16):
    """Infinite X elements in columns without blocks never meet a padding weight; X and Y are
    windows of wider tensors, at an odd column offset (fp32) or an even one (bf16)."""
    T, N, K = 230, 1032, 768
    M = matrix(N, K, R, C, 0.9, 7, False)
    X, _ = inputs(T, K, 7, False)
    # Free one block-column of blocks: rebuild without it.
    dense = host(B.bsr_to_dense(M))
    dense[:, :C] = 0.0
    nz = int((np.abs(dense.reshape(N // R, R, K // C, C)).max((1, 3)) > 0).sum())
    M = B.bsr_prune_from_dense(dev(dense), R, C, k=nz)
    assert not (host(M.indices)[:nz] == 0).any()
    assert_enough_work(M, T, bf16)
    if bf16:
        M = M.to_bf16()
    Xw = X.copy()
    Xw[:, :C] = np.inf
    off = 2 if bf16 else 1
    big = torch.zeros((T, K + 10), device="cuda:0")
    big[:, off:off + K] = dev(Xw)
    if bf16:
        big = B.bsr_cast_f32_bf16(big)
    Yb = torch.full((T, N + 5), 7.0, device="cuda:0")
    log(f"mtile inf/pitch {R}x{C} {'bf16' if bf16 else 'f32'}")
    B.bsr_spmm(big[:, off:off + K], M, None, Yb[:, 3:3 + N])
    X[:, :C] = 0.0
    check_spmm(X, M, None, Yb[:, 3:3 + N], bf16=bf16)
    assert bool((Yb[:, :3] == 7.0).all()) and bool((Yb[:, 3 + N:] == 7.0).all())


def check_batch(products, dense, kernel=None, slices=None, seed=0):
    """A batched call's outputs (Y filled with NaN before) against the oracle on sampled tokens."""
    for _, _, _, Y in products:
        Y.fill_(float("nan"))
    B.bsr_spmm_batched(products, kernel=kernel, slices=slices)
    g = np.random.Generator(np.random.PCG64(seed))
    for (Xd, M, bias, Y), X in zip(products, dense):
        assert bool(torch.isfinite(Y).all()), "outputs were not written"
        rows = np.unique(np.r_[0, X.shape[0] - 1, g.integers(0, X.shape[0], 40)])
        check_spmm(X, M, host(bias), Y, rows=rows, bf16=M.data.dtype == torch.bfloat16)


# Layers whose plan needs other slices than the launch's automatic (None) or asked-for count, as the
# launch's search and the one-slice search visit different counts.
SLICES = [(8, 8, 1024, 1256, 2560, 0.05, None, False), (4, 4, 1120, 1256, 2560, 0.05, None, False),
          (8, 1, 896, 1268, 2560, 0.05, None, False), (8, 8, 1024, 1256, 2560, 0.3, None, False),
          (8, 8, 256, 19720, 700, 0.05, None, True), (8, 8, 32, 20000, 700, 0.5, 3, False),
          (8, 1, 32, 20160, 700, 0.5, 3, False), (8, 8, 32, 20000, 700, 0.5, 5, False)]


@pytest.mark.parametrize("case", range(len(SLICES)))
def test_mtile_slices_of_the_launch(device, case):
    """Alone and beside another product of the launch, whatever the slice count."""
    R, C, N, K, T, d, slices, bf16 = SLICES[case]
    log(f"mtile launch slices {R}x{C} {'bf16' if bf16 else 'f32'} {N}x{K} T={T} d={d} S={slices}")
    products, dense = [], []
    for i, (n, k) in enumerate([(N, K), (768, 768)]):
        M = matrix(n, k, R, C, d, 30 + i, False)
        X, Xd = inputs(T, k, 30 + i, bf16)
        products.append((Xd, M.to_bf16() if bf16 else M, dev(np.linspace(-1, 1, n).astype(np.float32)),
                         torch.empty((T, n), device="cuda:0")))
        dense.append(X)
    check_batch(products[:1], dense, slices=slices)
    check_batch(products, dense, slices=slices)
    check_batch(products[::-1], dense[::-1], slices=slices)


# Feed-forward pairs of a 768-wide layer: the second product's input is staged in column chunks.
#   T, layers as (N, K), density.
BATCHES = [(777, [(3072, 768), (768, 3072)], 0.2),           # bf16: one launch, staged stores off
           (4096, [(3072, 768), (768, 3072)], 0.1),          # two launches, one of each kind
           (4001, [(768, 3072), (768, 768), (1032, 768), (768, 3072)], 0.15),
           (2051, [(768, 768), (1024, 1024)], 0.3)]          # staged stores fit one product only


@pytest.mark.parametrize("bf16", [False, True], ids=["f32", "bf16"])
@pytest.mark.parametrize("R,C", [(8, 8), (4, 4)], ids=["8x8", "4x4"])
@pytest.mark.parametrize("case", range(len(BATCHES)))
def test_mtile_batched(device, case, R, C, bf16):
    """Several products in one call: whole-row and column-chunked ones in a launch or split over two,
    against the oracle, and bit for bit against the generic kernel for integer inputs.  A timed call's
    events span all launches."""
    T, layers, d = BATCHES[case]
    log(f"mtile batch {R}x{C} {'bf16' if bf16 else 'f32'} T={T} {layers} d={d}")
    products, dense, ints = [], [], []
    for i, (n, k) in enumerate(layers):
        M = matrix(n, k, R, C, d, 50 + i, i == 0)
        assert_enough_work(M, T, bf16)
        X, Xd = inputs(T, k, 50 + i, bf16)
        bias = dev(np.linspace(-1, 1, n).astype(np.float32))
        products.append((Xd, M.to_bf16() if bf16 else M, bias, torch.empty((T, n), device="cuda:0")))
        dense.append(X)
        M = matrix(n, k, R, C, d, 50 + i, i == 0, integer=True)
        ints.append((inputs(T, k, 50 + i, bf16, integer=True)[1], M.to_bf16() if bf16 else M, None,
                     torch.full((T, n), float("nan"), device="cuda:0")))
    check_batch(products, dense, seed=case)
    B.bsr_spmm_batched(ints)
    for Xd, M, _, Y in ints:
        assert torch.equal(Y, B.bsr_spmm_ex(Xd, M, None, None, kernel=B.KERNEL_GENERIC))
    call = B.SpmmBatchCall(products)
    want = [Y.clone() for Y in call()]
    start, stop = (torch.cuda.Event(enable_timing=True) for _ in range(2))
    start.record()
    stop.record()
    for Y in call.Y:
        Y.zero_()
    call.timed(start, stop)
    stop.synchronize()
    assert start.elapsed_time(stop) > 0.0
    assert all(torch.equal(a, b) for a, b in zip(want, call.Y)), "not reproducible"
