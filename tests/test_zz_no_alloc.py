"""lrbi_masked_gemm_static (the entry point that allocates nothing: partial sums in the library's own static
scratch array) against lrbi_masked_gemm with a caller workspace, through the C ABI: identical bits, on two
calls in a row, the second with a smaller input that leaves part of the first call's scratch contents behind."""
import ctypes

import numpy as np
import pytest
import torch

import paper_1905_05686_amd as lrbi
import workloads
from oracle import lrbi_oracle as orc
from gpu_util import TOL, desc_of, dev, device_factors, to_device, workspace_for
from test_dispatch import geom, given, plan

pytestmark = pytest.mark.gpu

DC = {"f32": lrbi.F32, "f16": lrbi.F16, "bf16": lrbi.BF16}


def _case(cfg):
    data = workloads.make(cfg)
    d = desc_of(cfg)
    dIp, dIz = device_factors(d, data["Ip01"], data["Iz01"])
    W = to_device(data["W"], cfg.dtype)
    X = to_device(data["X"], cfg.dtype)
    return data, d, dIp, dIz, W, X


def _both(cfg):
    data, d, dIp, dIz, W, X = _case(cfg)
    need = lrbi.masked_gemm_workspace_bytes(d, DC[cfg.dtype], cfg.N)
    ws = workspace_for(d, DC[cfg.dtype], cfg.N)
    ref = lrbi.masked_gemm(d, W, dIp, dIz, X, workspace=ws)
    out = torch.full_like(ref, float("nan"))
    torch.cuda.synchronize()
    before = torch.cuda.memory_allocated()
    lrbi.masked_gemm_static(d, W, dIp, dIz, X, out)
    torch.cuda.synchronize()
    assert torch.cuda.memory_allocated() == before
    assert torch.equal(out.view(torch.int16 if out.element_size() == 2 else torch.int32),
                       ref.view(torch.int16 if ref.element_size() == 2 else torch.int32)), cfg
    # and, like every product, against the oracle
    M = orc.decode_mask(data["Ip01"], data["Iz01"], cfg.m, cfg.n, cfg.r, cfg.c, cfg.k)
    Y = orc.masked_gemm(workloads.to_float64(data["W"], cfg.dtype), M, workloads.to_float64(data["X"], cfg.dtype),
                        threads=16)
    assert orc.rel_err(out.double().cpu().numpy(), Y) <= TOL[cfg.dtype]
    return need


def test_two_calls_in_a_row_second_smaller():
    print("no-alloc: C2-shaped split product, then a smaller one", flush=True)
    big = workloads.Config("na-big", 2048, 4608, 256, 256, 16, 0.08, 128, "f16", 0.01, 5)     # split over n: scratch used
    small = workloads.Config("na-small", 512, 2048, 128, 128, 8, 0.2, 32, "bf16", 0.03, 6)    # split, fewer planes
    need_big = _both(big)
    need_small = _both(small)
    assert need_big > need_small > 0, (need_big, need_small)
    # a shape that needs no scratch at all goes straight through
    assert _both(workloads.Config("na-none", 512, 512, 128, 128, 8, 0.2, 2048, "bf16", 0.03, 7)) == 0


def test_sizes_beyond_the_scratch_are_refused_before_any_launch():
    # a forced split into 8 slices of 16384 x 128 fp32 partial sums: 64 MiB, beyond the 32 MiB array
    d = lrbi.Desc(16384, 8192, 256, 256, 16, lrbi.flag_splitk(8))
    assert lrbi.masked_gemm_workspace_bytes(d, lrbi.F16, 128) > lrbi.STATIC_SCRATCH_BYTES
    lib = lrbi.load_library()
    p = ctypes.c_void_p(256)     # never dereferenced: the size check comes before any launch
    assert lib.lrbi_masked_gemm_static(ctypes.byref(d), lrbi.F16, p, 8192, p, p, p, 128, 128, p, 128, None) == -8
    assert "workspace" in lrbi.strerror(-8)


def test_many_tiles_beyond_the_scratch_run_unsplit():
    """264 output tiles whose slices would need more than the scratch array: the bits of a call without a workspace."""
    cfg = workloads.Config("t", 4100, 2056, 256, 256, 16, 0.08, 1024, "f16", 0.03, 3)
    print("static scratch, many tiles", cfg, flush=True)
    _, d, dIp, dIz, W, X = _case(cfg)
    assert lrbi.masked_gemm_workspace_bytes(d, lrbi.F16, cfg.N) > 32 * 1024 * 1024
    ref = lrbi.masked_gemm(d, W, dIp, dIz, X)
    out = torch.full_like(ref, float("nan"))
    lrbi.masked_gemm_static(d, W, dIp, dIz, X, out)
    torch.cuda.synchronize()
    assert torch.equal(out.view(torch.int16), ref.view(torch.int16))
    split = lrbi.masked_gemm(d, W, dIp, dIz, X, workspace=workspace_for(d, lrbi.F16, cfg.N))
    torch.cuda.synchronize()
    assert orc.rel_err(split.double().cpu().numpy(), ref.double().cpu().numpy()) <= 1e-3  # f16 roundings of fp32 sums


def test_many_tiles_leave_the_scratch_alone():
    """264 output tiles whose slices would fit the scratch array: unsplit all the same, so that two such calls share nothing."""
    cfg = workloads.Config("t", 4100, 2056, 256, 256, 16, 0.08, 1000, "f16", 0.03, 3)
    print("static scratch, many tiles that fit", cfg, flush=True)
    _, d, dIp, dIz, W, X = _case(cfg)
    assert 0 < lrbi.masked_gemm_workspace_bytes(d, lrbi.F16, cfg.N) <= 32 * 1024 * 1024
    ref = lrbi.masked_gemm(d, W, dIp, dIz, X)
    split = lrbi.masked_gemm(d, W, dIp, dIz, X, workspace=workspace_for(d, lrbi.F16, cfg.N))
    out = torch.full_like(ref, float("nan"))
    lrbi.masked_gemm_static(d, W, dIp, dIz, X, out)
    torch.cuda.synchronize()
    assert not torch.equal(split, ref)  # the slices add up in another order
    assert torch.equal(out.view(torch.int16), ref.view(torch.int16))


def test_many_tiles_whose_slices_would_fit_run_unsplit():
    """The same on a batch that only the general kernel takes, whose plan with a workspace does have slices."""
    cfg = workloads.Config("t", 4100, 2056, 256, 256, 16, 0.08, 1004, "f16", 0.03, 3)
    print("static scratch, slices that would fit", cfg, flush=True)
    p = plan(geom(4100, 2056, 256, 256, 16), 1004, False)
    assert p.split_optional and p.splitk > 1 and p.workspace_bytes <= 32 * 1024 * 1024
    _, d, dIp, dIz, W, X = _case(cfg)
    ref = lrbi.masked_gemm(d, W, dIp, dIz, X)
    split = lrbi.masked_gemm(d, W, dIp, dIz, X, workspace=workspace_for(d, lrbi.F16, cfg.N))
    out = torch.full_like(ref, float("nan"))
    lrbi.masked_gemm_static(d, W, dIp, dIz, X, out)
    torch.cuda.synchronize()
    assert not torch.equal(split, ref)  # the slices add up in another order
    assert torch.equal(out.view(torch.int16), ref.view(torch.int16))


def test_decoded_mask_behind_the_planes_of_the_scratch():
    """Shapes whose mask is decoded first: planes and mask in the static array, two calls in a row, the second smaller."""
    print("static scratch, mask behind the planes", flush=True)
    for m, N in ((1200, 512), (900, 264)):
        p = given(geom(m, 3000, 300, 300, 8), N)
        assert p.splitk > 1 and p.workspace_bytes + m * 384 <= 32 * 1024 * 1024
        assert _both(workloads.Config("na-mask", m, 3000, 300, 300, 8, 0.2, N, "bf16", 0.03, 8)) >= p.workspace_bytes + m * 384


def test_decoded_mask_that_the_scratch_has_no_room_for():
    """A mask of 40 MB: the bits of a call with a workspace of the array's size, which rebuilds the mask in the kernel."""
    m, n, r, c, k, N = 20000, 16000, 500, 500, 8, 40
    print("static scratch, mask too large", (m, n, r, c, k, N), flush=True)
    p = given(geom(m, n, r, c, k), N)
    assert p is not None and m * 2000 > 32 * 1024 * 1024
    d = lrbi.Desc(m, n, r, c, k)
    gen = torch.Generator(device=dev()).manual_seed(9)

    def words(shape, valid):  # about one bit in four of the valid ones set
        draw = lambda: torch.randint(-2 ** 31, 2 ** 31, shape, dtype=torch.int32, device=dev(), generator=gen)  # noqa: E731
        left = (valid - 32 * torch.arange(shape[1], device=dev())).clamp(0, 32)
        return draw() & draw() & torch.where(left == 32, -1, (1 << left) - 1).to(torch.int32)
    ip, iz = words((d.tiles * r, 1), k), words((d.tiles * k, 16), c)
    W = torch.randn((m, n), device=dev(), generator=gen).half()
    X = torch.randn((n, N), device=dev(), generator=gen).half()
    ref = lrbi.masked_gemm(d, W, ip, iz, X, workspace=torch.empty(lrbi.STATIC_SCRATCH_BYTES, dtype=torch.uint8, device=dev()))
    first = lrbi.masked_gemm(d, W, ip, iz, X, workspace=workspace_for(d, lrbi.F16, N))
    out = torch.full_like(ref, float("nan"))
    lrbi.masked_gemm_static(d, W, ip, iz, X, out)
    torch.cuda.synchronize()
    assert torch.equal(out.view(torch.int16), ref.view(torch.int16))
    assert not torch.equal(first.view(torch.int16), ref.view(torch.int16))
    assert orc.rel_err(first.double().cpu().numpy(), ref.double().cpu().numpy()) <= 1e-3  # f16 roundings of fp32 sums
