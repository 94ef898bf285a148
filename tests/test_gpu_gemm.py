"""GPU parity: lrbi_masked_gemm against the fp64 CPU oracle."""
import numpy as np
import pytest
import torch

import paper_1905_05686_amd as lrbi
import workloads
from oracle import lrbi_oracle as orc
from gpu_util import (ORACLE_THREADS, TOL, TORCH_DTYPE, desc_of, dev, device_factors, to_device, to_float64,
                      unpack_device_mask, workspace_for)
from test_dispatch import PIPE, PIPE256, geom, given, plan

pytestmark = pytest.mark.gpu

DT_CODE = {"f32": lrbi.F32, "f16": lrbi.F16, "bf16": lrbi.BF16}


def _run(cfg, data, flags=0, use_workspace=True, ldpad=0):
    desc = desc_of(cfg, flags)
    dIp, dIz = device_factors(desc, data["Ip01"], data["Iz01"])
    W = to_device(data["W"], cfg.dtype)
    X = to_device(data["X"], cfg.dtype)
    if ldpad:
        Wp = torch.zeros((cfg.m, cfg.n + ldpad), dtype=W.dtype, device=dev())
        Wp[:, :cfg.n] = W
        W = Wp[:, :cfg.n]
        Xp = torch.zeros((cfg.n, cfg.N + ldpad), dtype=X.dtype, device=dev())
        Xp[:, :cfg.N] = X
        X = Xp[:, :cfg.N]
    ws = workspace_for(desc, DT_CODE[cfg.dtype], cfg.N) if use_workspace else None
    Y = lrbi.masked_gemm(desc, W, dIp, dIz, X, workspace=ws)
    torch.cuda.synchronize()
    return Y


def _oracle(cfg, data):
    M = orc.decode_mask(data["Ip01"], data["Iz01"], cfg.m, cfg.n, cfg.r, cfg.c, cfg.k)
    return orc.masked_gemm(workloads.to_float64(data["W"], cfg.dtype), M, workloads.to_float64(data["X"], cfg.dtype),
                           threads=ORACLE_THREADS), M


def _assert_close(Y, ref, dtype, what=""):
    err = orc.rel_err(to_float64(Y), ref)
    normwise = float(np.max(np.abs(to_float64(Y) - ref)) / max(np.max(np.abs(ref)), 1e-300))
    print("%s rel_err %.3e (normwise %.3e, tol %.0e)" % (what, err, normwise, TOL[dtype]), flush=True)
    assert err <= TOL[dtype], (what, err)


@pytest.mark.parametrize("name", ["C1", "C2", "C3a", "C3b", "C4", "C5"])
def test_config_parity(name):
    cfg = workloads.CONFIGS[name]
    print("gemm config", name, flush=True)
    data = workloads.make(cfg)
    ref, _ = _oracle(cfg, data)
    Y = _run(cfg, data)
    _assert_close(Y, ref, cfg.dtype, name)
    # run-to-run identical bits (no floating-point atomics anywhere)
    Y2 = _run(cfg, data)
    assert torch.equal(Y.view(torch.int16 if Y.element_size() == 2 else torch.int32),
                       Y2.view(torch.int16 if Y.element_size() == 2 else torch.int32))


def _small(m, n, r, c, k, p, N, dtype, seed=0, sigma=0.05):
    return workloads.Config("t", m, n, r, c, k, p, N, dtype, sigma, seed)


EDGE = [
    # shape                                         forced flags
    (_small(96, 200, 48, 100, 4, 0.2, 1, "f32"), 0),
    (_small(96, 200, 48, 100, 4, 0.2, 7, "f32"), 0),
    (_small(33, 77, 3, 7, 3, 0.3, 2, "f32"), 0),             # nothing aligned: scalar loads everywhere
    (_small(130, 4104, 65, 1368, 9, 0.1, 1, "bf16"), lrbi.FLAG_PATH_VALU),  # n spans three 2048-column segments
    (_small(130, 4104, 65, 1368, 9, 0.1, 3, "f16"), 0),
    (_small(128, 192, 64, 64, 8, 0.2, 128, "bf16"), 0),      # one 128x128 tile, 3 slabs
    (_small(300, 2400, 300, 300, 8, 0.12, 20, "f16"), lrbi.FLAG_PATH_MFMA),  # unaligned tiles, scalar X path, split
    (_small(3000, 600, 300, 300, 8, 0.12, 20, "f16"), 0),    # the row-streaming kernel by itself: 190 workgroups, the last of a tile row with 12 rows
    (_small(2100, 512, 300, 128, 6, 0.15, 8, "bf16"), 0),    # the same, bf16, 7 tile rows of 19 workgroups
    (_small(384, 1024, 128, 256, 16, 0.1, 72, "f16"), 0),    # 128x64 tile variant (N in 33..64 -> padded)
    (_small(384, 1024, 128, 256, 16, 0.1, 40, "bf16"), 0),
    (_small(384, 1024, 128, 256, 16, 0.1, 48, "bf16"), lrbi.FLAG_PATH_MFMA | lrbi.flag_tile(10)),  # the 128 x 64 panel kernel by flag
    (_small(384, 1024, 128, 256, 16, 0.1, 44, "f16"), 0),    # N no multiple of 8: the 128 x 64 panel kernel by itself
    (_small(200, 1000, 100, 500, 40, 0.05, 136, "bf16"), 0), # rank above 32, ragged m and N
    (_small(256, 2048, 128, 512, 32, 0.06, 256, "bf16"), lrbi.FLAG_PATH_MFMA | lrbi.flag_splitk(4)),
    (_small(256, 2048, 128, 512, 32, 0.06, 256, "f16"), lrbi.FLAG_PATH_MFMA | lrbi.flag_splitk(1)),
    (_small(256, 512, 128, 128, 8, 0.2, 2, "f16"), lrbi.FLAG_PATH_MFMA),   # tiny batch forced onto MFMA
    (_small(256, 512, 128, 128, 8, 0.2, 64, "bf16"), lrbi.FLAG_PATH_VALU), # big batch forced onto the ALUs
    (_small(256, 512, 128, 128, 8, 0.2, 96, "bf16"), lrbi.FLAG_PATH_MFMA | lrbi.flag_tile(2)),
    (_small(256, 512, 128, 128, 8, 0.2, 96, "bf16"), lrbi.FLAG_PATH_MFMA | lrbi.flag_tile(3)),
    # tile shape and ranks of the paper's own experiments (Sec. 4: 576 x 512 tiles, rank 145; Table 1: rank 256)
    (_small(1152, 1024, 576, 512, 145, 0.02, 64, "f16"), 0),
    (_small(1152, 1024, 576, 512, 256, 0.015, 1, "bf16"), 0),
    (_small(64, 576, 64, 576, 8, 0.2, 12416, "bf16"), 0),    # few rows, many columns: 64-column blocks, unsplit
    (_small(48, 288, 16, 96, 4, 0.3, 3080, "f16"), 0),       # ... 32-column blocks
    (_small(4096, 2304, 256, 256, 16, 0.08, 3, "bf16"), 0),  # three columns of a large matrix: the tile kernel, mostly idle
    # few rows, short rows: the row-streaming kernels on a grid far smaller than the chip (automatic choice)
    (_small(1200, 600, 1200, 600, 145, 0.05, 20, "f16"), 0), # the gate matrix of an LSTM layer of size 300 (Sec. 4), untiled, at Table 2's rank 145
    (_small(800, 400, 800, 400, 145, 0.05, 20, "f16"), 0),   # 50 workgroups
    (_small(128, 1024, 128, 256, 16, 0.1, 8, "f16"), 0),     # eight workgroups
    (_small(64, 4096, 64, 256, 16, 0.1, 1, "bf16"), 0),      # eight workgroups of the single-column kernel
    # tile widths that are an odd multiple of 64 on the pipelined tile kernel (Table 2's 576-column tiles): 128-column
    # units of the mask that lie across two tile columns
    (_small(256, 1152, 128, 576, 8, 0.2, 128, "f16"), 0),      # two tile columns, three panels, the last one short
    (_small(256, 3456, 128, 576, 40, 0.05, 136, "bf16"), 0),   # two I_p words per row, two column blocks, ragged N
    (_small(128, 9216, 128, 576, 32, 0.054, 128, "f16"), 0),   # split over n: slices begin inside tiles
    (_small(256, 768, 256, 192, 16, 0.1, 72, "bf16"), 0),      # 192-column tiles
    (_small(128, 512, 128, 64, 8, 0.2, 128, "f16"), 0),        # 64-column tiles: every unit has two tiles
    (_small(256, 1152, 128, 576, 8, 0.2, 64, "f16"), 0),       # 33 to 64 columns on these widths: the same kernel, half a block
    (_small(256, 1152, 128, 576, 8, 0.2, 40, "bf16"), 0),
    (_small(256, 2304, 128, 576, 16, 0.1, 256, "bf16"), lrbi.FLAG_PATH_MFMA | lrbi.flag_splitk(3)),
]


@pytest.mark.parametrize("idx", range(len(EDGE)))
def test_edge_shapes(idx):
    cfg, flags = EDGE[idx]
    print("gemm edge", idx, cfg, hex(flags), flush=True)
    data = workloads.make(cfg)
    ref, _ = _oracle(cfg, data)
    _assert_close(_run(cfg, data, flags=flags), ref, cfg.dtype, "edge%d" % idx)


# The row-streaming kernel (narrow batches), forced so that small matrices take it too; the configurations C3a and
# C4 above reach it on their own.
STREAM = [
    _small(100, 200, 50, 100, 4, 0.2, 1, "bf16"),        # last workgroup has 4 of its 16 rows, one short slab
    _small(130, 4104, 65, 1368, 9, 0.1, 4, "f16"),       # 16 slabs and 8 columns; tiles cut through slabs and words
    _small(300, 2400, 300, 300, 8, 0.12, 20, "f16"),     # C4's tiles and batch
    _small(256, 512, 128, 128, 8, 0.2, 32, "bf16"),      # both 16-column blocks full
    _small(48, 264, 24, 33, 5, 0.3, 8, "f16"),           # tiles narrower than two mask words
    _small(1152, 1024, 576, 512, 145, 0.02, 16, "f16"),  # rank 145: five I_p words per row
    _small(64, 520, 32, 130, 6, 0.25, 12, "bf16"),
    _small(64, 520, 32, 130, 6, 0.25, 28, "f16"),
    _small(2048, 8, 512, 8, 2, 0.5, 1, "f16"),           # a single 16-byte piece per row
    _small(64, 96, 32, 32, 3, 0.3, 8, "bf16"),           # a tile row's I_z is no whole number of 16-byte pieces
    # one column: a row travels in registers (rows of up to 8192 columns; 2, 4, 8 or 16 pieces of 1 KB)
    _small(130, 4104, 65, 1368, 9, 0.1, 1, "bf16"),      # 16 pieces, the ninth holds 8 columns; tiles cut through words
    _small(64, 4096, 32, 512, 32, 0.1, 1, "f16"),        # 8 full pieces
    _small(72, 8192, 24, 1024, 16, 0.08, 1, "bf16"),     # 16 full pieces
    _small(1152, 1024, 576, 512, 145, 0.02, 1, "f16"),   # 2 pieces, rank 145
    _small(44, 1544, 22, 772, 7, 0.2, 1, "f16"),         # 4 pieces, the last one short; 6 of 8 rows in the last workgroup
    _small(40, 8704, 20, 1088, 6, 0.15, 1, "bf16"),      # longer rows: back on the staged kernel, 17 slabs of 512
]


@pytest.mark.parametrize("idx", range(len(STREAM)))
def test_row_streaming_kernel(idx):
    cfg = STREAM[idx]
    print("gemm stream", idx, cfg, flush=True)
    data = workloads.make(cfg)
    ref, M = _oracle(cfg, data)
    Y = _run(cfg, data, flags=lrbi.FLAG_PATH_STREAM)
    _assert_close(Y, ref, cfg.dtype, "stream%d" % idx)
    # nothing stored under a pruned bit reaches Y, also not through the clamped loads past the last row and column
    W = workloads.to_float64(data["W"], cfg.dtype).astype(np.float32)
    poison = np.where(np.arange(cfg.n)[None, :] % 2 == 0, np.nan, np.inf).astype(np.float32)
    data["W"] = workloads.to_storage(np.where(M == 1, W, poison), cfg.dtype)
    Yp = _run(cfg, data, flags=lrbi.FLAG_PATH_STREAM)
    assert torch.equal(Y.view(torch.int16), Yp.view(torch.int16))


def test_row_streaming_kernel_refuses_what_it_cannot_serve():
    cfg = _small(64, 520, 32, 130, 6, 0.25, 6, "f16")  # N = 6: neither 1 nor a multiple of 4
    data = workloads.make(cfg)
    with pytest.raises(lrbi.LrbiError):
        _run(cfg, data, flags=lrbi.FLAG_PATH_STREAM)
    cfg = _small(64, 520, 32, 130, 6, 0.25, 1, "f32")
    with pytest.raises(lrbi.LrbiError):
        _run(cfg, workloads.make(cfg), flags=lrbi.FLAG_PATH_STREAM)


@pytest.mark.parametrize("dtype,N", [("bf16", 1), ("f16", 20)])
def test_row_streaming_identity_x_returns_masked_weights_exactly(dtype, N):
    cfg = _small(256, 256, 128, 128, 8, 0.2, N, dtype)
    data = workloads.make(cfg)
    X = np.zeros((cfg.n, N), np.float32)
    X[np.arange(N), np.arange(N)] = 1.0
    data["X"] = workloads.to_storage(X, dtype)
    M = orc.decode_mask(data["Ip01"], data["Iz01"], cfg.m, cfg.n, cfg.r, cfg.c, cfg.k)
    Wm = np.where(M == 1, workloads.to_float64(data["W"], dtype), 0.0)
    Y = to_float64(_run(cfg, data, flags=lrbi.FLAG_PATH_STREAM))
    assert np.array_equal(Y, Wm[:, :N])


def test_padded_leading_dimensions():
    for cfg in (_small(128, 256, 64, 128, 8, 0.2, 24, "f16"), _small(128, 256, 64, 128, 8, 0.2, 1, "bf16"),
                _small(50, 120, 25, 60, 4, 0.2, 3, "f32")):
        for pad in (8, 3):
            print("gemm ldpad", cfg.dtype, cfg.N, pad, flush=True)
            data = workloads.make(cfg)
            ref, _ = _oracle(cfg, data)
            _assert_close(_run(cfg, data, ldpad=pad), ref, cfg.dtype, "ldpad")


def test_without_workspace_falls_back_to_unsplit_kernel():
    cfg = _small(300, 2400, 300, 300, 8, 0.12, 20, "f16")
    data = workloads.make(cfg)
    assert lrbi.masked_gemm_workspace_bytes(desc_of(cfg), lrbi.F16, cfg.N) > 0
    ref, _ = _oracle(cfg, data)
    _assert_close(_run(cfg, data, flags=lrbi.FLAG_PATH_MFMA, use_workspace=False), ref, cfg.dtype, "no-ws")
    with pytest.raises(lrbi.LrbiError) as e:
        _run(cfg, data, flags=lrbi.FLAG_PATH_MFMA | lrbi.flag_splitk(2), use_workspace=False)
    assert e.value.status == -8


@pytest.mark.parametrize("dtype,N", [("f16", 256), ("bf16", 256), ("bf16", 1), ("f32", 1), ("f16", 20)])
def test_identity_x_returns_masked_weights_exactly(dtype, N):
    # X = [I | 0]: Y[:, q] = (W o M)[:, q] bit for bit, which isolates the masking
    cfg = _small(256, 256, 128, 128, 8, 0.2, N, dtype)
    data = workloads.make(cfg)
    X = np.zeros((cfg.n, N), np.float32)
    X[np.arange(min(N, cfg.n)), np.arange(min(N, cfg.n))] = 1.0
    data["X"] = workloads.to_storage(X, dtype)
    M = orc.decode_mask(data["Ip01"], data["Iz01"], cfg.m, cfg.n, cfg.r, cfg.c, cfg.k)
    Wm = np.where(M == 1, workloads.to_float64(data["W"], dtype), 0.0)
    Y = to_float64(_run(cfg, data))
    assert np.array_equal(Y, Wm[:, :N])


@pytest.mark.parametrize("dtype,N", [("f16", 128), ("bf16", 128), ("bf16", 1), ("f32", 2)])
def test_values_under_pruned_bits_never_reach_y(dtype, N):
    cfg = _small(256, 512, 128, 256, 8, 0.15, N, dtype)
    data = workloads.make(cfg)
    ref, M = _oracle(cfg, data)
    W = workloads.to_float64(data["W"], dtype).astype(np.float32)
    poison = np.where(np.arange(cfg.n)[None, :] % 2 == 0, np.nan, np.inf).astype(np.float32)
    W = np.where(M == 1, W, poison)
    data["W"] = workloads.to_storage(W, dtype)
    Y = _run(cfg, data)
    assert torch.isfinite(Y).all()
    _assert_close(Y, ref, dtype, "poison")


@pytest.mark.parametrize("dtype", ["f16", "bf16"])
def test_output_rounding_is_nearest_even(dtype):
    # small integers: every product and partial sum is exact in fp32, so the only rounding
    # is the final one, which must be round-to-nearest-even of the exact result
    cfg = _small(128, 512, 128, 256, 8, 0.3, 128, dtype)
    rng = np.random.default_rng(5)
    data = workloads.make(cfg)
    data["W"] = workloads.to_storage(rng.integers(-8, 9, (cfg.m, cfg.n)).astype(np.float32), dtype)
    data["X"] = workloads.to_storage(rng.integers(-8, 9, (cfg.n, cfg.N)).astype(np.float32), dtype)
    ref, _ = _oracle(cfg, data)
    assert np.abs(ref).max() > 256  # beyond bf16's exact-integer range, so rounding really happens
    exp = workloads.to_float64(workloads.to_storage(ref, dtype), dtype)
    Y = to_float64(_run(cfg, data))
    assert np.array_equal(Y, exp)


def test_all_ones_factors_equal_dense_product():
    cfg = _small(256, 512, 128, 128, 4, 1.0, 128, "bf16")
    data = workloads.make(cfg)
    assert data["Ip01"].all() and data["Iz01"].all()
    Y = _run(cfg, data)
    ref = workloads.to_float64(data["W"], "bf16") @ workloads.to_float64(data["X"], "bf16")
    _assert_close(Y, ref, "bf16", "dense")
    zero = dict(data, Ip01=data["Ip01"] * 0)
    assert not to_float64(_run(cfg, zero)).any()


def test_full_size_sampled_rows_in_bench_configuration():
    """C2 at full size in the launch configuration bench.py times, checked on rows the
    oracle computes one by one (independent of test_config_parity's whole-matrix check)."""
    cfg = workloads.CONFIGS["C2"]
    data = workloads.make(cfg)
    Y = to_float64(_run(cfg, data))
    Wd = workloads.to_float64(data["W"], cfg.dtype)
    Xd = workloads.to_float64(data["X"], cfg.dtype)
    tile_cols = cfg.n // cfg.c
    rng = np.random.default_rng(3)
    rms = float(np.sqrt(np.mean(Y * Y)))
    for i in [0, cfg.m - 1] + [int(v) for v in rng.integers(cfg.m, size=30)]:
        ti, il = divmod(i, cfg.r)
        row = np.zeros(cfg.N)
        for tj in range(tile_cols):
            t = ti * tile_cols + tj
            bits = orc.decode_mask(data["Ip01"][t:t + 1, il:il + 1], data["Iz01"][t:t + 1], 1, cfg.c, 1, cfg.c, cfg.k)
            row += orc.masked_gemm(Wd[i:i + 1, tj * cfg.c:(tj + 1) * cfg.c], bits, Xd[tj * cfg.c:(tj + 1) * cfg.c])[0]
        err = np.max(np.abs(Y[i] - row) / np.maximum(np.abs(row), rms))
        assert err <= TOL[cfg.dtype], (i, err)


# ---- mask and product from one call (rows a1-a6 fused)
FUSED = [
    _small(256, 1152, 128, 128, 8, 0.2, 128, "f16"),     # the tile kernel leaves the mask: one column block, unsplit
    _small(256, 1024, 256, 256, 16, 0.1, 256, "bf16"),   # two column blocks: only the first one stores the mask
    _small(256, 1024, 256, 256, 16, 0.1, 48, "bf16"),    # 33 to 64 columns: the same kernel, part of its column block idle
    _small(128, 9216, 128, 256, 16, 0.08, 128, "f16"),   # split over n: every slice stores its own units, last panel short
    (_small(300, 2400, 300, 300, 8, 0.12, 20, "f16"), lrbi.FLAG_PATH_MFMA),  # generic tile kernel, 32-column blocks, tiles cut through mask words
    _small(1200, 600, 1200, 600, 145, 0.05, 20, "f16"),  # few, short rows (an LSTM layer of size 300 at rank 145): the ring kernel on 75 workgroups
    _small(130, 264, 65, 33, 5, 0.3, 70, "bf16"),        # generic tile kernel, tiles narrower than two mask words
    _small(260, 520, 128, 128, 8, 0.2, 96, "f16"),       # generic kernel on cut-off aligned tiles: 8 bits of the last piece live
    _small(1152, 1024, 576, 512, 145, 0.02, 64, "f16"),  # rank 145
    _small(256, 1088, 128, 64, 8, 0.2, 200, "bf16"),     # two blocks of columns, n a multiple of 64 but not of 128
    _small(50, 120, 25, 60, 4, 0.2, 3, "f32"),
    workloads.CONFIGS["C2"],                             # the benchmark's workload at full size
    # the pipelined tile kernel on tile widths of 64 (2 j + 1): mask units gathered per 64-column half
    _small(256, 1152, 128, 576, 8, 0.2, 128, "f16"),
    _small(256, 3456, 128, 576, 40, 0.05, 136, "bf16"),
    _small(128, 9216, 128, 576, 32, 0.054, 128, "f16"),
    _small(128, 512, 128, 64, 8, 0.2, 128, "f16"),
    _small(256, 1152, 128, 576, 8, 0.2, 40, "bf16"),
    workloads.Config("paper_fc5_tiles", 4096, 9216, 512, 576, 32, 0.054, 128, "f16", 0.01),  # Table 2's tiling of C2's layer
    # narrow batches with enough rows for the row-streaming kernels: they store the rows' mask from LDS
    _small(3000, 600, 300, 300, 8, 0.12, 20, "f16"),     # ring kernel, tiles cut through mask words, last workgroups short
    _small(2048, 1024, 256, 128, 8, 0.15, 1, "bf16"),    # single-column kernel
    _small(1040, 4104, 65, 1368, 9, 0.1, 1, "bf16"),     # single-column kernel, n no multiple of 128: the last piece's pad bits
    _small(1040, 8704, 520, 1088, 6, 0.15, 1, "bf16"),   # one column over rows longer than 8192: the ring kernel's 8-row form
    workloads.CONFIGS["C3a"],
    workloads.CONFIGS["C4"],
]


@pytest.mark.parametrize("N", [1, 8, 128])
def test_fp16_subnormal_weights_are_not_flushed(N):
    """Weights below fp16's smallest normal number (2^-14) times inputs of 2^10: exact in fp32, and far above zero in
    the sum; a path that flushes subnormal operands (the 2-element dot products of the single-column kernel, the
    matrix cores of the others) would return zeros."""
    cfg = _small(128, 1024, 128, 256, 8, 0.3, N, "f16")
    rng = np.random.default_rng(11)
    data = workloads.make(cfg)
    data["W"] = (rng.integers(1, 64, (cfg.m, cfg.n)).astype(np.float32) * np.float32(2.0 ** -24)).astype(np.float16)
    data["X"] = np.full((cfg.n, cfg.N), 1024.0, dtype=np.float16)
    ref, M = _oracle(cfg, data)
    assert np.abs(ref).max() > 1e-3 and M.sum() > 0
    Y = to_float64(_run(cfg, data))
    # every product k * 2^-14 and every partial sum is exact in fp32; only the final rounding to fp16 is left
    exp = workloads.to_float64(workloads.to_storage(ref, "f16"), "f16")
    assert np.array_equal(Y, exp)


@pytest.mark.parametrize("idx", range(len(FUSED)))
def test_decode_and_gemm_equals_the_two_calls(idx):
    cfg, flags = FUSED[idx] if isinstance(FUSED[idx], tuple) else (FUSED[idx], 0)
    print("decode_and_gemm", idx, cfg, hex(flags), flush=True)
    data = workloads.make(cfg)
    desc = desc_of(cfg, flags)
    dIp, dIz = device_factors(desc, data["Ip01"], data["Iz01"])
    W, X = to_device(data["W"], cfg.dtype), to_device(data["X"], cfg.dtype)
    ws = workspace_for(desc, DT_CODE[cfg.dtype], cfg.N)
    pitch = ((cfg.n + 127) // 128) * 16 + 32
    mask = torch.full((cfg.m, pitch), 0xA5, dtype=torch.uint8, device=dev())
    mask2 = torch.full((cfg.m, pitch), 0xA5, dtype=torch.uint8, device=dev())
    m1, Y1 = lrbi.decode_and_gemm(desc, W, dIp, dIz, X, mask=mask, workspace=ws)
    lrbi.decode_mask(desc, dIp, dIz, out=mask2)
    Y2 = lrbi.masked_gemm(desc, W, dIp, dIz, X, workspace=ws)
    torch.cuda.synchronize()
    assert torch.equal(m1, mask2)  # the bytes beyond the written part of a row are left alone by both
    assert torch.equal(Y1.view(torch.uint8), Y2.view(torch.uint8))
    # and against the oracle
    M = orc.decode_mask(data["Ip01"], data["Iz01"], cfg.m, cfg.n, cfg.r, cfg.c, cfg.k)
    assert np.array_equal(unpack_device_mask(m1, cfg.n)[:, :cfg.n], M)
    ref, _ = _oracle(cfg, data)
    _assert_close(Y1, ref, cfg.dtype, "fused%d" % idx)


@pytest.mark.parametrize("m,n,r,c,k,N,ldpad", [
    (33, 65, 11, 13, 3, 5, 0),         # scalar loads, one row and one column past the blocks
    (500, 800, 100, 100, 4, 64, 0),    # a thirteenth chunk of columns
    (70, 516, 35, 129, 40, 33, 4),     # two I_p words, four columns in the last chunk, padded rows
    (8200, 72, 200, 72, 4, 70, 0),     # two batch blocks per workgroup, the last one short
    (8200, 71, 200, 71, 4, 64, 0),
])
def test_fp32_batches(m, n, r, c, k, N, ldpad):
    """fp32 products of five columns and more against the fp64 oracle; fp32 sums of up to 800 terms in chunks."""
    cfg = workloads.Config("t", m, n, r, c, k, 0.25, N, "f32", 0.05, 5)
    print("fp32 batch", cfg, ldpad, flush=True)
    data = workloads.make(cfg)
    d = desc_of(cfg)
    dIp, dIz = device_factors(d, data["Ip01"], data["Iz01"])
    W = torch.zeros((m, n + ldpad), device=dev())
    W[:, :n] = to_device(data["W"], "f32")
    M = orc.decode_mask(data["Ip01"], data["Iz01"], m, n, r, c, k)
    ref = orc.masked_gemm(data["W"].astype(np.float64), M, data["X"].astype(np.float64))
    Y = lrbi.masked_gemm(d, W[:, :n], dIp, dIz, to_device(data["X"], "f32"))
    torch.cuda.synchronize()
    assert orc.rel_err(Y.double().cpu().numpy(), ref) <= 1e-6


@pytest.mark.parametrize("m,n,r,c,k,p,N", [
    (260, 328, 200, 192, 40, 0.25, 72),    # rows with more than eight set ranks, two I_p words, cut-off tiles
    (130, 64, 100, 64, 3, 0.3, 40),       # one slab: nothing lies ahead
    (129, 200, 43, 128, 33, 0.2, 33),     # an odd number of slabs, N not in whole pieces
    (600, 4104, 150, 64, 16, 0.1, 128),   # slices; every slab in another tile
    (300, 960, 100, 320, 70, 0.05, 136),  # three I_p words: the words of a slab loaded at once
    (1100, 2056, 100, 100, 4, 0.3, 6),    # 32-column form: nine tiles, six slices
])
def test_general_tile_kernel_masks(m, n, r, c, k, p, N):
    """The general tile kernel's mask words, loaded ahead of their slab: mask bits exact, product against the oracle."""
    cfg = workloads.Config("t", m, n, r, c, k, p, N, "f16", 0.05, 11)
    print("general tile kernel", cfg, flush=True)
    data = workloads.make(cfg)
    d = desc_of(cfg)
    dIp, dIz = device_factors(d, data["Ip01"], data["Iz01"])
    M = orc.decode_mask(data["Ip01"], data["Iz01"], m, n, r, c, k)
    ref = orc.masked_gemm(workloads.to_float64(data["W"], "f16"), M, workloads.to_float64(data["X"], "f16"))
    mask, Y = lrbi.decode_and_gemm(d, to_device(data["W"], "f16"), dIp, dIz, to_device(data["X"], "f16"),
                                   workspace=workspace_for(d, lrbi.F16, N))
    torch.cuda.synchronize()
    bits = unpack_device_mask(mask, n)
    assert np.array_equal(bits[:, :n], M) and not bits[:, n:].any()
    assert orc.rel_err(to_float64(Y), ref) <= TOL["f16"]


@pytest.mark.parametrize("m,n,r,c,k,N", [
    (64, 576, 64, 64, 8, 5),        # 16 wavefronts, seven of them without a second chunk
    (65, 1100, 33, 100, 5, 40),     # scalar loads; a last chunk of 12 columns
    (64, 16384, 64, 256, 8, 6),     # long rows, few of them: vector ALUs up to six columns
    (64, 16384, 64, 256, 8, 7),
    (4100, 520, 100, 104, 4, 8),    # 129 workgroups: eight wavefronts again
])
def test_fp32_batches_of_few_rows(m, n, r, c, k, N):
    """fp32 products around the lines between the forms of the kernel, against the fp64 oracle."""
    test_fp32_batches(m, n, r, c, k, N, 0)


# 256 x 256 tiles: one slab panel and several, tile rows that change inside a workgroup's rows, an odd number of 128-row
# blocks, half units of two tiles, one and two I_p words, column blocks cut off at N, tile groups that are not full
@pytest.mark.parametrize("m,n,r,c,k,N,dtype", [
    (128, 64, 128, 64, 5, 8, "bf16"),
    (256, 128, 256, 128, 32, 256, "f16"),
    (384, 576, 128, 192, 33, 264, "f16"),
    (512, 1024, 256, 512, 64, 248, "bf16"),
    (640, 1152, 128, 576, 32, 520, "bf16"),
    (1408, 320, 128, 64, 16, 1032, "f16"),
])
def test_tiles_of_256(m, n, r, c, k, N, dtype):
    print("256 x 256 tiles", m, n, r, c, k, N, dtype, flush=True)
    cfg = workloads.Config("t256", m, n, r, c, k, 0.12, N, dtype, 0.05)
    data = workloads.make(cfg)
    ref, _ = _oracle(cfg, data)
    for ldpad in (0, 8):
        Y = _run(cfg, data, flags=lrbi.flag_tile(15), ldpad=ldpad)
        _assert_close(Y, ref, dtype, "256 x 256")
    # the sums are formed per accumulator in the order of the columns in either form, but in other groups: close, not equal
    Y2 = _run(cfg, data, flags=lrbi.flag_tile(14))
    _assert_close(Y2, ref, dtype, "128 x 128")
    assert torch.equal(Y, _run(cfg, data, flags=lrbi.flag_tile(15), ldpad=8))


# the pipelined kernel on matrices that end inside a tile: last rows, last slab and last panel cut at every kind of place, one
# tile larger than the matrix, half units, split and not, the mask stored as well, junk in what cut-off tiles do not use
@pytest.mark.parametrize("m,n,r,c,k,N,dtype", [
    (260, 520, 128, 128, 8, 96, "f16"),
    (127, 8, 128, 64, 5, 40, "bf16"),
    (129, 72, 256, 64, 33, 136, "f16"),
    (300, 1096, 128, 192, 40, 64, "bf16"),
    (513, 2312, 256, 576, 16, 128, "f16"),
    (255, 632, 256, 1024, 9, 72, "bf16"),
    (384, 576, 128, 192, 12, 264, "f16"),
    (4100, 520, 512, 256, 16, 1032, "bf16"),
])
def test_pipelined_kernel_on_cut_off_tiles(m, n, r, c, k, N, dtype):
    print("pipelined kernel, cut-off tiles", m, n, r, c, k, N, dtype, flush=True)
    cfg = workloads.Config("rag", m, n, r, c, k, 0.12, N, dtype, 0.05)
    data = workloads.make(cfg)
    ref, M = _oracle(cfg, data)
    for ldpad in (0, 8):
        for use_workspace in (True, False):
            _assert_close(_run(cfg, data, use_workspace=use_workspace, ldpad=ldpad), ref, dtype, "cut off")
    # factors packed as for whole tiles: bits outside the matrix are there and must be ignored
    desc = desc_of(cfg)
    ip, iz = lrbi.pack_factors(lrbi.Desc(-(-m // r) * r, -(-n // c) * c, r, c, k), data["Ip01"], data["Iz01"])
    dIp, dIz = torch.from_numpy(ip.view(np.int32)).to(dev()), torch.from_numpy(iz.view(np.int64)).to(dev())
    mask = torch.full((m, 16 * ((n + 127) // 128) + 16), 0x5A, dtype=torch.uint8, device=dev())
    out, Y = lrbi.decode_and_gemm(desc, to_device(data["W"], dtype), dIp, dIz, to_device(data["X"], dtype), mask=mask,
                                  workspace=workspace_for(desc, DT_CODE[dtype], N))
    torch.cuda.synchronize()
    _assert_close(Y, ref, dtype, "cut off, mask stored")
    bits = unpack_device_mask(out, n)
    used = 128 * ((n + 127) // 128)
    assert np.array_equal(bits[:, :n], M) and not bits[:, n:used].any()
    assert (out.cpu().numpy()[:, used // 8:] == 0x5A).all()


# tile shapes that line up with nothing and ranks above 64, more than 32 columns: the mask decoded first, behind the planes of
# the workspace or in the caller's own buffer, then the pipelined kernel on it; without a workspace the general kernel
@pytest.mark.parametrize("m,n,r,c,k,N,dtype", [
    (1200, 3000, 300, 300, 8, 512, "bf16"),
    (1153, 2048, 576, 512, 145, 136, "f16"),
    (1000, 1992, 100, 100, 33, 264, "bf16"),
    (4100, 1096, 192, 83, 5, 520, "f16"),
])
def test_pipelined_kernel_on_a_decoded_mask(m, n, r, c, k, N, dtype):
    print("pipelined kernel, decoded mask", m, n, r, c, k, N, dtype, flush=True)
    cfg = workloads.Config("given", m, n, r, c, k, 0.12 if k < 64 else 0.03, N, dtype, 0.05)
    data = workloads.make(cfg)
    ref, M = _oracle(cfg, data)
    for ldpad in (0, 8):
        for use_workspace in (True, False):
            _assert_close(_run(cfg, data, use_workspace=use_workspace, ldpad=ldpad), ref, dtype, "decoded mask")
    desc = desc_of(cfg)
    dIp, dIz = device_factors(desc, data["Ip01"], data["Iz01"])
    W, X = to_device(data["W"], dtype), to_device(data["X"], dtype)
    ws = workspace_for(desc, DT_CODE[dtype], N)
    mask, Y = lrbi.decode_and_gemm(desc, W, dIp, dIz, X, workspace=ws)
    torch.cuda.synchronize()
    _assert_close(Y, ref, dtype, "mask wanted")
    assert np.array_equal(unpack_device_mask(mask, n)[:, :n], M)
    # a pruned weight never reaches the sum, whatever it holds
    Wn = torch.where(torch.from_numpy(M.astype(bool)).to(dev()), W, torch.full_like(W, float("nan")))
    assert torch.equal(lrbi.masked_gemm(desc, Wn, dIp, dIz, X, workspace=ws), lrbi.masked_gemm(desc, W, dIp, dIz, X, workspace=ws))


def test_decoded_mask_with_rows_far_apart():
    """Rows of the caller's mask more than 2^32 / 127 bytes apart: a lane's 32-bit offset does not reach the tile's last rows."""
    m, n, r, c, k, N = 128, 3000, 300, 300, 8, 4096
    pitch = 33818656  # 127 rows further lies 2016 bytes past 2^32
    print("mask rows %d bytes apart" % pitch, flush=True)
    cfg = workloads.Config("far", m, n, r, c, k, 0.12, N, "f16", 0.05)
    data = workloads.make(cfg)
    ref, M = _oracle(cfg, data)
    desc = desc_of(cfg)
    dIp, dIz = device_factors(desc, data["Ip01"], data["Iz01"])
    mask = torch.empty((m, pitch), dtype=torch.uint8, device=dev())
    ws = workspace_for(desc, lrbi.F16, N)
    out, Y = lrbi.decode_and_gemm(desc, to_device(data["W"], "f16"), dIp, dIz, to_device(data["X"], "f16"), mask=mask, workspace=ws)
    torch.cuda.synchronize()
    assert np.array_equal(unpack_device_mask(out[:, :16 * ((n + 127) // 128)], n)[:, :n], M)
    _assert_close(Y, ref, "f16", "far rows")


# the 256 x 256 form (which does not store the mask), tiles that line up with nothing (the mask decoded first, if the workspace
# has room for it), cut-off tiles, the general kernel
@pytest.mark.parametrize("m,n,r,c,k,N", [
    (4096, 128, 128, 64, 8, 4096),
    (1200, 3000, 300, 300, 8, 512),
    (1290, 1096, 128, 192, 40, 264),
    (300, 960, 100, 64, 33, 100),
])
def test_mask_and_product_in_one_call_have_the_bits_of_two(m, n, r, c, k, N):
    cfg = workloads.Config("both", m, n, r, c, k, 0.12, N, "bf16", 0.05)
    print("mask and product in one call", cfg, flush=True)
    data = workloads.make(cfg)
    desc = desc_of(cfg)
    dIp, dIz = device_factors(desc, data["Ip01"], data["Iz01"])
    W, X = to_device(data["W"], "bf16"), to_device(data["X"], "bf16")
    ref_mask = lrbi.decode_mask(desc, dIp, dIz)
    asked = lrbi.masked_gemm_workspace_bytes(desc, lrbi.BF16, N)
    for nbytes in (asked, asked - ref_mask.numel(), 0):  # (without room for a mask)
        ws = torch.empty(nbytes, dtype=torch.uint8, device=dev()) if nbytes > 0 else None
        ref = lrbi.masked_gemm(desc, W, dIp, dIz, X, workspace=ws)
        for pad in (0, 16):
            mask = torch.empty((m, ref_mask.shape[1] + pad), dtype=torch.uint8, device=dev())
            mask, Y = lrbi.decode_and_gemm(desc, W, dIp, dIz, X, mask=mask, workspace=ws)
            torch.cuda.synchronize()
            assert torch.equal(mask[:, :ref_mask.shape[1]], ref_mask)
            assert torch.equal(Y.view(torch.int16), ref.view(torch.int16)), (nbytes, pad)


# infinities in the last row of X where the last slab of 64 columns is cut off: a kept weight carries them to Y as infinities, as on
# the general kernel (a pruned one meets them as zero: NaN); nothing but the last row itself may be multiplied with them
@pytest.mark.parametrize("m,n,r,c,k,N,tile", [
    (127, 8, 128, 64, 5, 40, 14), (260, 520, 128, 128, 8, 96, 14), (300, 1096, 128, 192, 40, 64, 14), (255, 632, 256, 1024, 9, 72, 14),
    (513, 2312, 256, 576, 16, 128, 0), (1200, 3000, 300, 300, 8, 512, 0), (640, 1992, 100, 100, 33, 1032, 0),
])
def test_infinities_in_the_last_row_of_x(m, n, r, c, k, N, tile):
    cfg = workloads.Config("inf", m, n, r, c, k, 0.3, N, "f16", 0.05)
    print("infinities in the last row of X", cfg, "tile", tile, flush=True)
    data = workloads.make(cfg)
    M = orc.decode_mask(data["Ip01"], data["Iz01"], m, n, r, c, k)
    X = data["X"].copy()
    X[n - 1, ::3] = np.inf
    X[n - 1, 1::3] = -np.inf
    with np.errstate(invalid="ignore"):
        ref = (workloads.to_float64(data["W"], "f16") * M) @ workloads.to_float64(X, "f16")
    assert np.isinf(ref).any() and np.isnan(ref).any()
    desc = desc_of(cfg, lrbi.flag_tile(tile))
    dIp, dIz = device_factors(desc, data["Ip01"], data["Iz01"])
    W, dX = to_device(data["W"], "f16"), to_device(X, "f16")
    ws = workspace_for(desc, lrbi.F16, N)
    for Y in (lrbi.masked_gemm(desc, W, dIp, dIz, dX, workspace=ws), lrbi.decode_and_gemm(desc, W, dIp, dIz, dX, workspace=ws)[1]):
        torch.cuda.synchronize()
        Y = to_float64(Y)
        assert np.array_equal(np.isnan(Y), np.isnan(ref))
        assert np.array_equal(np.where(np.isinf(Y), Y, 0), np.where(np.isinf(ref), ref, 0))
        ok = np.isfinite(ref)
        assert orc.rel_err(np.where(ok, Y, 0), np.where(ok, ref, 0)) <= TOL["f16"]


def _product_and_mask(cfg, data, flags=0):
    """Y from either entry point against the oracle, the stored mask against it bit for bit."""
    m, n, N = cfg.m, cfg.n, cfg.N
    ref, M = _oracle(cfg, data)
    desc = desc_of(cfg, flags)
    dIp, dIz = device_factors(desc, data["Ip01"], data["Iz01"])
    W, X = to_device(data["W"], cfg.dtype), to_device(data["X"], cfg.dtype)
    for ws in (workspace_for(desc, DT_CODE[cfg.dtype], N), None):
        _assert_close(lrbi.masked_gemm(desc, W, dIp, dIz, X, workspace=ws), ref, cfg.dtype, "product")
        mask, Y = lrbi.decode_and_gemm(desc, W, dIp, dIz, X, workspace=ws)
        torch.cuda.synchronize()
        _assert_close(Y, ref, cfg.dtype, "mask stored")
        bits = unpack_device_mask(mask, n)
        assert np.array_equal(bits[:, :n], M) and not bits[:, n:].any()


# sizes of the pipelined kernel's cut-off form that its own rule leaves to another one: the smallest input (one slab of eight
# columns), two-word half units over several panels, more than 256 tiles with a cut-off last row block
@pytest.mark.parametrize("m,n,r,c,k,N,dtype", [
    (127, 8, 128, 64, 5, 40, "bf16"),
    (300, 1096, 128, 192, 40, 64, "bf16"),
    (4100, 520, 512, 256, 16, 1032, "bf16"),
    (130, 1544, 128, 320, 64, 8, "f16"),
])
def test_cut_off_tiles_forced_on_the_pipelined_kernel(m, n, r, c, k, N, dtype):
    print("pipelined kernel asked for, cut-off tiles", m, n, r, c, k, N, dtype, flush=True)
    g = geom(m, n, r, c, k)
    assert plan(g, N, True).tile != PIPE and plan(g, N, True, lrbi.flag_tile(PIPE)).tile == PIPE
    cfg = workloads.Config("rag", m, n, r, c, k, 0.12, N, dtype, 0.05)
    _product_and_mask(cfg, workloads.make(cfg), lrbi.flag_tile(PIPE))


# ... and sizes that reach a form by the rules
@pytest.mark.parametrize("m,n,r,c,k,N,tile", [
    (4096, 128, 128, 64, 8, 4096, PIPE256),
    (3968, 384, 128, 192, 33, 4088, PIPE256),
    (513, 2312, 256, 576, 16, 128, PIPE),
    (1152, 2048, 576, 512, 145, 136, None),  # None: the mask decoded first
    (1153, 2056, 576, 512, 145, 904, None),
    (520, 3000, 100, 100, 33, 1064, None),
])
def test_forms_that_the_rules_choose(m, n, r, c, k, N, tile):
    print("form chosen by the rules", m, n, r, c, k, N, tile, flush=True)
    g = geom(m, n, r, c, k)
    assert (given(g, N) is not None) if tile is None else (given(g, N) is None and plan(g, N, True).tile == tile)
    cfg = workloads.Config("rule", m, n, r, c, k, 0.12 if k < 64 else 0.03, N, "f16", 0.05)
    _product_and_mask(cfg, workloads.make(cfg))
