"""GPU parity of the backward pass through the masking layer (Sec. 2): lrbi_masked_gemm_t (dX = (W o I_a)^T dY) and
lrbi_masked_grad (dW = (dY X^T) o I_a) against the fp64 oracle."""
import numpy as np
import pytest
import torch

import paper_1905_05686_amd as lrbi
import workloads
from oracle import lrbi_oracle as orc
from gpu_util import TOL, desc_of, dev, device_factors, to_device, to_float64

pytestmark = pytest.mark.gpu

DT_CODE = {"f32": lrbi.F32, "f16": lrbi.F16, "bf16": lrbi.BF16}


def _inputs(cfg):
    data = workloads.make(cfg)
    rng = np.random.default_rng(cfg.seed + 77)
    dY = workloads.to_storage(rng.standard_normal((cfg.m, cfg.N), dtype=np.float32), cfg.dtype)
    return data, dY


def _padded(t, pad):
    if not pad:
        return t
    p = torch.zeros((t.shape[0], t.shape[1] + pad), dtype=t.dtype, device=t.device)
    p[:, :t.shape[1]] = t
    return p[:, :t.shape[1]]


def _check(cfg, ldpad=0, use_workspace=True, what=""):
    print("backward", what, cfg, "ldpad", ldpad, flush=True)
    data, dYs = _inputs(cfg)
    desc = desc_of(cfg)
    dIp, dIz = device_factors(desc, data["Ip01"], data["Iz01"])
    W = _padded(to_device(data["W"], cfg.dtype), ldpad)
    X = _padded(to_device(data["X"], cfg.dtype), ldpad)
    dY = _padded(to_device(dYs, cfg.dtype), ldpad)
    ws = None
    nbytes = lrbi.masked_gemm_t_workspace_bytes(desc, DT_CODE[cfg.dtype], cfg.N)
    if use_workspace and nbytes:
        ws = torch.empty(nbytes // 4, dtype=torch.float32, device=dev())
    dX = lrbi.masked_gemm_t(desc, W, dIp, dIz, dY, workspace=ws)
    dW = lrbi.masked_grad(desc, dY, X, dIp, dIz)
    torch.cuda.synchronize()
    M = orc.decode_mask(data["Ip01"], data["Iz01"], cfg.m, cfg.n, cfg.r, cfg.c, cfg.k)
    W64, X64, dY64 = (workloads.to_float64(a, cfg.dtype) for a in (data["W"], data["X"], dYs))
    e1 = orc.rel_err(to_float64(dX), orc.masked_gemm_t(W64, M, dY64))
    dW_ref = orc.masked_grad(dY64, X64, M)
    dWh = to_float64(dW)
    e2 = orc.rel_err(dWh, dW_ref)
    print("dX rel_err %.3e  dW rel_err %.3e (tol %.0e)" % (e1, e2, TOL[cfg.dtype]), flush=True)
    assert e1 <= TOL[cfg.dtype] and e2 <= TOL[cfg.dtype]
    assert not dWh[M == 0].any(), "pruned weights must get exactly zero"
    # identical bits from call to call
    dX2 = lrbi.masked_gemm_t(desc, W, dIp, dIz, dY, workspace=ws)
    dW2 = lrbi.masked_grad(desc, dY, X, dIp, dIz)
    view = torch.int16 if dX.element_size() == 2 else torch.int32
    assert torch.equal(dX.view(view), dX2.view(view)) and torch.equal(dW.view(view), dW2.view(view))
    return dX, dW


@pytest.mark.parametrize("name", ["C1", "C2", "C3b", "C4", "C5"])
def test_config_parity(name):
    _check(workloads.CONFIGS[name], what=name)


def _small(m, n, r, c, k, p, N, dtype, seed=0):
    return workloads.Config("t", m, n, r, c, k, p, N, dtype, 0.05, seed)


EDGE = [
    (_small(10, 10, 5, 5, 2, 0.5, 1, "f32"), 0),
    (_small(96, 200, 48, 100, 4, 0.2, 7, "f32"), 3),
    (_small(33, 77, 3, 7, 3, 0.3, 9, "bf16"), 0),               # nothing aligned: vector-ALU kernels
    (_small(256, 256, 128, 128, 8, 0.2, 64, "f16"), 0),
    (_small(640, 256, 128, 128, 8, 0.2, 24, "bf16"), 0),        # narrow batch tile, split over m
    (_small(300, 1096, 128, 256, 8, 0.15, 72, "f16"), 0),       # edge tiles
    (_small(130, 200, 65, 100, 40, 0.05, 136, "bf16"), 8),      # padded leading dimensions, rank above 32
    (_small(200, 136, 100, 136, 4, 0.3, 20, "f16"), 0),         # N not a multiple of 8
    (_small(1152, 1024, 576, 512, 145, 0.02, 128, "bf16"), 0),  # the paper's tile shape and a rank it uses
    (_small(768, 256, 384, 128, 40, 0.05, 16, "bf16"), 0),      # slices that start inside a tile, two I_p words
    (_small(1024, 384, 256, 384, 16, 0.1, 40, "f16"), 0),       # workgroups at three offsets inside a tile column
    (_small(512, 128, 128, 128, 64, 0.03, 8, "f16"), 0),        # smallest tile rows of the tuned mask path, rank 64
    (_small(2048, 512, 512, 512, 32, 0.06, 4, "bf16"), 0),      # batch of 4: the tile kernel's 32-column form, mostly idle
    (_small(1024, 640, 256, 128, 16, 0.1, 1, "f16"), 0),        # one column
    (_small(300, 1096, 128, 256, 8, 0.15, 3, "bf16"), 0),       # three columns, edge tiles
    # the pipelined transposed kernel (aligned tiles, batch above 32 columns)
    (_small(256, 256, 128, 128, 8, 0.2, 128, "f16"), 0),        # one panel of four slabs, one 128-row unit per tile row
    (_small(1536, 384, 256, 384, 16, 0.1, 136, "bf16"), 0),     # three panels, three slices, a short second batch block
    (_small(1024, 128, 128, 128, 64, 0.03, 72, "f16"), 0),      # rank 64: two I_p words per row, a batch block of 72
    (_small(768, 256, 384, 128, 40, 0.05, 80, "bf16"), 8),      # rank 40, three units per tile row, padded leading dimensions
    (_small(2048, 256, 512, 256, 5, 0.3, 256, "f16"), 0),       # rank 5 (a short round of ranks), four panels
    (_small(1024, 256, 256, 128, 16, 0.1, 48, "bf16"), 0),      # 33 to 64 batch columns: part of the batch block idle
    # the same kernel on tile widths that are an odd multiple of 64 (Table 2's 576-column tiles): workgroups whose 128
    # columns lie in two tile columns
    (_small(512, 1152, 128, 576, 8, 0.2, 128, "f16"), 0),       # nine workgroups, the fifth across the two tile columns
    (_small(1536, 1152, 512, 576, 40, 0.05, 136, "bf16"), 0),   # two I_p words, three panels, slices, a short batch block
    (_small(1024, 384, 256, 192, 16, 0.1, 72, "f16"), 8),       # 192-column tiles, padded leading dimensions
    (_small(640, 256, 128, 64, 8, 0.2, 128, "bf16"), 0),        # 64-column tiles: every workgroup has two tile columns
    (_small(2048, 1152, 512, 576, 64, 0.04, 256, "f16"), 0),    # rank 64, four panels
    (_small(256, 960, 128, 192, 8, 0.2, 24, "f16"), 0),         # gradient: the last column block's upper half is past the matrix
    (_small(1024, 1152, 512, 576, 32, 0.054, 64, "bf16"), 0),   # gradient: rank 32 on 576-column tiles
]


@pytest.mark.parametrize("idx", range(len(EDGE)))
def test_edge_shapes(idx):
    cfg, ldpad = EDGE[idx]
    _check(cfg, ldpad=ldpad)


def test_without_workspace_the_reduction_is_not_split():
    cfg = _small(2048, 256, 128, 128, 8, 0.2, 32, "f16")
    assert lrbi.masked_gemm_t_workspace_bytes(desc_of(cfg), lrbi.F16, cfg.N) > 0
    a, _ = _check(cfg, use_workspace=True)
    b, _ = _check(cfg, use_workspace=False)
    assert orc.rel_err(to_float64(a), to_float64(b)) <= 1e-2


@pytest.mark.parametrize("N", [16, 128])
def test_nonfinite_values_under_pruned_weights_never_reach_dx(N):
    cfg = _small(256, 512, 128, 256, 8, 0.15, N, "f16")
    data, dYs = _inputs(cfg)
    desc = desc_of(cfg)
    M = orc.decode_mask(data["Ip01"], data["Iz01"], cfg.m, cfg.n, cfg.r, cfg.c, cfg.k)
    Wn = data["W"].copy()
    Wn[M == 0] = np.float16(np.nan)
    Wn[::3][M[::3] == 0] = np.float16(np.inf)
    dIp, dIz = device_factors(desc, data["Ip01"], data["Iz01"])
    dY = to_device(dYs, cfg.dtype)
    a = lrbi.masked_gemm_t(desc, to_device(data["W"], cfg.dtype), dIp, dIz, dY)
    b = lrbi.masked_gemm_t(desc, to_device(Wn, cfg.dtype), dIp, dIz, dY)
    torch.cuda.synchronize()
    assert torch.equal(a.view(torch.int16), b.view(torch.int16))


@pytest.mark.parametrize("cfg,ldpad", [
    (_small(1, 1, 1, 1, 1, 1.0, 1, "f32"), 0),
    (_small(65, 33, 20, 33, 3, 0.4, 33, "f32"), 0),             # one row, one column past the blocks; scalar loads
    (_small(520, 96, 104, 48, 33, 0.05, 64, "f32"), 4),         # a ninth chunk of rows, two I_p words, padded leading dimensions
    (_small(1030, 4100, 206, 82, 4, 0.2, 132, "f32"), 0),       # two blocks per workgroup, the last one short
    (_small(64, 9000, 32, 250, 4, 0.3, 40, "f32"), 0),          # one chunk of rows; two blocks per workgroup
    (_small(64, 301, 64, 301, 4, 0.3, 20, "bf16"), 0),          # one chunk of rows, 16-bit
    (_small(130, 77, 65, 11, 4, 0.3, 40, "f16"), 0),            # 16-bit rows that are not whole pieces
    (_small(70, 8300, 35, 83, 4, 0.3, 70, "bf16"), 0),          # the same, two batch blocks per workgroup
])
def test_fp32_matrix_cores(cfg, ldpad):
    _check(cfg, ldpad=ldpad, what="fp32 instructions")


@pytest.mark.parametrize("m", [200, 64])                # 64: a chunk of rows, one wavefront in the transposed product
@pytest.mark.parametrize("N", [1, 4, 5, 33, 50, 64, 97])  # one sweep below 5; one, 18 and 32 columns in a last block
def test_fp32_products_with_nonfinite_operands(N, m):
    """An infinity or a NaN in the batch reaches the results of kept weights only, in both products."""
    cfg = _small(m, 168, 50, 56, 4, 0.3, N, "f32")
    print("nonfinite batch", N, flush=True)
    data, dY = _inputs(cfg)
    d = desc_of(cfg)
    dIp, dIz = device_factors(d, data["Ip01"], data["Iz01"])
    M = orc.decode_mask(data["Ip01"], data["Iz01"], cfg.m, cfg.n, cfg.r, cfg.c, cfg.k)
    X = data["X"].copy()
    X[3, 0], X[100, N - 1], dY[7, 0], dY[m - 1, N - 1] = np.inf, np.nan, -np.inf, np.nan
    W = to_device(data["W"], "f32")
    Y = lrbi.masked_gemm(d, W, dIp, dIz, to_device(X, "f32"))
    dX = lrbi.masked_gemm_t(d, W, dIp, dIz, to_device(dY, "f32"))
    torch.cuda.synchronize()
    for got, mask, bad in ((Y, M, X), (dX, M.T, dY)):
        reached = mask.astype(np.float64) @ (~np.isfinite(bad)).astype(np.float64) > 0
        assert np.array_equal(~np.isfinite(got.cpu().numpy()), reached)
    ok = [np.where(np.isfinite(a), a, 0).astype(np.float64) for a in (X, dY)]
    W64 = data["W"].astype(np.float64)
    for got, ref in ((Y, orc.masked_gemm(W64, M, ok[0])), (dX, orc.masked_gemm_t(W64, M, ok[1]))):
        h = got.cpu().numpy().astype(np.float64)
        fin = np.isfinite(h)
        assert orc.rel_err(np.where(fin, h, 0), np.where(fin, ref, 0)) <= TOL["f32"]


@pytest.mark.parametrize("transposed", [False, True])
def test_fp32_products_of_more_lanes_than_a_dimension_counts(transposed):
    """131073 blocks of rows (columns) x 65 of batch columns, 512 lanes each, are more than 2^32 lanes.  Rows from all over
    the result against float64."""
    size, red, N = 2 ** 22 + 1, 449, 4097
    print("fp32 product, many blocks, transposed", transposed, flush=True)
    gen = torch.Generator(device=dev())
    gen.manual_seed(9)
    dtype = torch.float16 if transposed else torch.float32
    X = torch.randn((red, N), device=dev(), generator=gen).to(dtype)
    W = torch.empty((red, size) if transposed else (size, red), dtype=dtype, device=dev()).normal_(0.0, 0.05, generator=gen)
    bits = lambda n: torch.randint(0, 2, (n,), dtype=torch.int32, device=dev(), generator=gen)
    pack = lambda b: (torch.nn.functional.pad(b, (0, -b.numel() % 64)).reshape(-1, 32) << torch.arange(32, device=dev(), dtype=torch.int32)).sum(
        1, dtype=torch.int32)
    m, n = W.shape
    ip, iz = bits(m), bits(n)  # rank 1, one tile
    got = (lrbi.masked_gemm_t if transposed else lrbi.masked_gemm)(lrbi.Desc(m, n, m, n, 1), W, ip[:, None].contiguous(), pack(iz)[None], X)
    torch.cuda.synchronize()
    rows = torch.cat([torch.randint(0, size, (500,), device=dev(), generator=gen), torch.arange(size - 40, size, device=dev())])
    Wr = (W.T[rows] if transposed else W[rows]).double()
    mask = (iz[rows, None] & ip[None]) if transposed else (ip[rows, None] & iz[None])
    ref = (Wr * mask) @ X.double()
    tol = 2.0 ** -10 if transposed else 1e-6  # the rounding of f16; fp32 sums of 449 terms in chunks
    assert float((got[rows].double() - ref).norm() / ref.norm()) <= tol
    assert torch.equal((got[rows] == 0).all(1), (mask == 0).all(1))


@pytest.mark.parametrize("long_side", ["m", "n"])
def test_nonfinite_operands_leave_the_finite_results_exact(long_side):
    """An infinity in the batch has its batch column formed again, the results it does not reach in sums in double: only
    the rounding to fp32 is left of their error, 2^-24 each.  The other columns hold the bits of a call without it."""
    cfg = _small(9000, 72, 250, 36, 3, 0.3, 20, "f32") if long_side == "m" else _small(72, 9000, 36, 250, 3, 0.3, 20, "f32")
    print("nonfinite, long side", long_side, flush=True)
    data, dY = _inputs(cfg)
    d = desc_of(cfg)
    dIp, dIz = device_factors(d, data["Ip01"], data["Iz01"])
    M = orc.decode_mask(data["Ip01"], data["Iz01"], cfg.m, cfg.n, cfg.r, cfg.c, cfg.k)
    W, W64 = to_device(data["W"], "f32"), data["W"].astype(np.float64)
    call, batch, mask, product = (lrbi.masked_gemm, data["X"], M, orc.masked_gemm) if long_side == "n" else \
        (lrbi.masked_gemm_t, dY, M.T, orc.masked_gemm_t)
    clean = call(d, W, dIp, dIz, to_device(batch, "f32")).cpu().numpy()
    bad = batch.copy()
    at = int(mask.sum(axis=0).argmax())
    bad[at, 3] = np.inf
    got = call(d, W, dIp, dIz, to_device(bad, "f32")).cpu().numpy()
    rest = [q for q in range(20) if q != 3]
    assert np.array_equal(got[:, rest].view(np.int32), clean[:, rest].view(np.int32))
    reached = mask[:, at] != 0
    assert np.array_equal(~np.isfinite(got[:, 3]), reached) and reached.any() and not reached.all()
    ref = product(W64, M, batch.astype(np.float64))[~reached, 3]
    assert orc.rel_err(got[~reached, 3].astype(np.float64), ref) <= 2.0 ** -24 * (1 + 1e-6)


# gradients in 256 x 256 tiles (rounds of 256 tiles nearly full from 128 batch columns, one round of 144 and more from 512): an
# odd number of 128-row blocks, a last column block cut off inside a half unit, two I_p words, half units of two tiles
@pytest.mark.parametrize("m,n,r,c,k,N,dtype", [
    (3968, 4032, 128, 64, 5, 128, "bf16"),
    (4096, 4032, 256, 576, 40, 160, "f16"),
    (2944, 3008, 128, 64, 64, 512, "bf16"),
])
def test_gradient_in_tiles_of_256(m, n, r, c, k, N, dtype):
    cfg = workloads.Config("g256", m, n, r, c, k, 0.15, N, dtype, 0.05)
    print("gradient, 256 x 256 tiles", cfg, flush=True)
    data, dYs = _inputs(cfg)
    desc = desc_of(cfg)
    dIp, dIz = device_factors(desc, data["Ip01"], data["Iz01"])
    M = orc.decode_mask(data["Ip01"], data["Iz01"], m, n, r, c, k)
    ref = orc.masked_grad(workloads.to_float64(dYs, dtype), workloads.to_float64(data["X"], dtype), M)
    for ldpad in (0, 8):
        X, dY = _padded(to_device(data["X"], dtype), ldpad), _padded(to_device(dYs, dtype), ldpad)
        dW = lrbi.masked_grad(desc, dY, X, dIp, dIz)
        dWh = to_float64(dW)
        assert orc.rel_err(dWh, ref) <= TOL[dtype]
        assert not dWh[M == 0].any(), "pruned weights must get exactly zero"
        assert torch.equal(dW.view(torch.int16), lrbi.masked_grad(desc, dY, X, dIp, dIz).view(torch.int16))


# mask words formed with four ranks at a time: windows that start before a tile's I_z row and end behind it, tiles narrower than a
# word, two and more I_p words, every rank set and none
@pytest.mark.parametrize("m,n,r,c,k,p,N,dtype", [
    (70, 90, 32, 9, 5, 1.0, 8, "f32"),
    (130, 200, 65, 33, 40, 0.5, 40, "f32"),
    (100, 264, 64, 100, 70, 0.1, 40, "bf16"),
    (96, 136, 50, 31, 3, 0.0, 16, "f16"),
])
def test_mask_words_four_ranks_at_a_time(m, n, r, c, k, p, N, dtype):
    _check(workloads.Config("ahead", m, n, r, c, k, p, N, dtype, 0.05, 3), what="mask words")
