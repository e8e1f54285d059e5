"""GPU parity of the weight compressor / decompressor / dense packer: bit-exact against the oracle."""
import ctypes
import gc

import numpy as np
import pytest
import torch

import oracle
from oracle import device_layout as dl
from paper_2411_00288_amd import binding, workloads as wl
from helpers import dev_bits, host_bits, layer_desc

pytestmark = pytest.mark.gpu

SHAPES = [  # cout, cin, kh, kw, korder
    (64, 64, 3, 3, wl.K_CRS),      # config-0 shape: K = 576 = 18 steps
    (256, 64, 1, 1, wl.K_CRS),
    (40, 8, 3, 3, wl.K_CRS),       # ragged rows (40 % 32), K = 72 (ragged step, odd step count)
    (7, 4, 1, 1, wl.K_CRS),        # a single block per row
    (96, 24, 2, 2, wl.K_RSC),      # K = 96 = 3 steps (odd: padded metadata half)
    (33, 96, 1, 1, wl.K_CRS),
    (130, 36, 3, 3, wl.K_RSC),     # K = 324: K % 32 = 4
    (1, 4, 1, 1, wl.K_CRS),
]


@pytest.mark.parametrize("shape", SHAPES)
@pytest.mark.parametrize("dtype", [wl.F16, wl.BF16])
@pytest.mark.parametrize("mask", ["logits", "top2"])
def test_packed_bytes_match_oracle_bit_for_bit(ss, shape, dtype, mask):
    cout, cin, kh, kw, korder = shape
    L = wl.Layer("t", N=1, H=4, W=4, cin=cin, cout=cout, kh=kh, kw=kw, dtype=dtype, korder=korder, mask=mask, seed=31)
    d = wl.make_inputs(L)
    Wb = d["W"].copy()
    special = [0x8000, 0x7E01, 0x7C00, 0x0001, 0xFC00, 0x8001, 0x0000, 0xFFFF]   # -0, NaN, inf, subnormals
    n = min(8, Wb.size)
    Wb.reshape(-1)[:n] = special[:n]
    desc = layer_desc(ss, L)
    assert ss.ss_packed_bytes(desc) == dl.packed_bytes(cout, L.K)
    W = dev_bits(Wb, dtype)
    M = torch.from_numpy(d["M"]).cuda()
    W_before, M_before = W.clone(), M.clone()
    packed = ss.ss_mask_compress(desc, W, M)
    vals, meta = oracle.compress(Wb, d["M"])
    expect = dl.tile(vals, meta, cin=cin, kh=kh, kw=kw, dtype=dtype, korder=korder)
    got = packed.cpu().numpy()
    assert got.size == expect.size
    assert np.array_equal(got, expect)
    # the inverse bijection recovers the canonical arrays from the GPU's bytes
    h, v2, m2 = dl.untile(got)
    assert np.array_equal(v2, vals) and np.array_equal(m2, meta)
    # inputs are never written (the original weights stay unchanged)
    assert torch.equal(W.view(torch.int16), W_before.view(torch.int16)) and torch.equal(M, M_before)
    # decompress gives M (.) W bit for bit, including the sign of kept zeros and NaN payloads
    back = host_bits(ss.ss_mask_decompress(desc, packed))
    assert np.array_equal(back, np.where(d["M"] == 1, Wb, 0).astype(np.uint16))
    assert np.array_equal(back, oracle.decompress(vals, meta))


def test_compress_reports_first_invalid_block(ss):
    L = wl.Layer("t", N=1, H=2, W=2, cin=16, cout=70, kh=3, kw=3, mask="logits", seed=1)
    d = wl.make_inputs(L)
    desc = layer_desc(ss, L)
    W = dev_bits(d["W"], L.dtype)
    for bad in ([(5, 7)], [(69, 35), (12, 0)], [(0, 0)], [(33, 20), (33, 3), (40, 1)]):
        Mb = d["M"].copy()
        for (r, g) in bad:
            Mb[r, 4 * g:4 * g + 4] = [1, 1, 1, 0]
        st, r0, g0 = oracle.mask_check(Mb)
        assert st == 1
        with pytest.raises(ss.SSError) as ei:
            ss.ss_mask_compress(desc, W, torch.from_numpy(Mb).cuda())
        assert ei.value.status == ss.SS_ERR_BAD_MASK
        assert ei.value.detail == (r0, g0) == min(bad)
    # a byte that is neither 0 nor 1 is rejected too
    Mb = d["M"].copy()
    Mb[3, 8:12] = [2, 0, 0, 0]
    with pytest.raises(ss.SSError) as ei:
        ss.ss_mask_compress(desc, W, torch.from_numpy(Mb).cuda())
    assert ei.value.detail == (3, 2)
    # all-zero and all-one blocks
    for fill in (0, 1):
        Mb = d["M"].copy()
        Mb[10, 0:4] = fill
        with pytest.raises(ss.SSError):
            ss.ss_mask_compress(desc, W, torch.from_numpy(Mb).cuda())


@pytest.mark.parametrize("shape", SHAPES + [(64, 3, 7, 7, wl.K_CRS), (5, 3, 3, 3, wl.K_RSC)])
@pytest.mark.parametrize("dtype", [wl.F16, wl.BF16])
def test_dense_pack_matches_oracle_layout(ss, shape, dtype):
    cout, cin, kh, kw, korder = shape
    K = cin * kh * kw
    masked = K % 4 == 0
    L = wl.Layer("t", N=1, H=8, W=8, cin=cin, cout=cout, kh=kh, kw=kw, dtype=dtype, korder=korder,
                 mask="logits" if masked else "none", seed=17)
    d = wl.make_inputs(L)
    desc = layer_desc(ss, L)
    assert ss.ss_dense_bytes(desc) == dl.dense_bytes(cout, K)
    W = dev_bits(d["W"], dtype)
    M = torch.from_numpy(d["M"]).cuda() if masked else None
    got = ss.ss_dense_pack(desc, W, M).cpu().numpy()
    Wm = np.where(d["M"] == 1, d["W"], 0).astype(np.uint16) if masked else d["W"]
    expect = dl.tile_dense(Wm, cin=cin, kh=kh, kw=kw, dtype=dtype, korder=korder)
    assert np.array_equal(got, expect)


def test_full_size_config1_compress(ss):
    L = wl.CONFIG1
    d = wl.make_inputs(wl.with_batch(L, 1))
    desc = layer_desc(ss, L)
    packed = ss.ss_mask_compress(desc, dev_bits(d["W"], L.dtype), torch.from_numpy(d["M"]).cuda())
    vals, meta = oracle.compress(d["W"], d["M"])
    expect = dl.tile(vals, meta, cin=L.cin, kh=L.kh, kw=L.kw, dtype=L.dtype, korder=L.korder)
    assert np.array_equal(packed.cpu().numpy(), expect)
    assert packed.numel() == 256 + 9 * (L.cout * L.K * 2) // 16


@pytest.mark.parametrize("shape", SHAPES)
@pytest.mark.parametrize("dtype", [wl.F16, wl.BF16])
def test_update_and_repack_match_oracle_bit_for_bit(ss, shape, dtype):
    """W <- round16(W + U), packed <- compress(W, M): both bit for bit (values chosen without NaN results)."""
    cout, cin, kh, kw, korder = shape
    L = wl.Layer("t", N=1, H=4, W=4, cin=cin, cout=cout, kh=kh, kw=kw, dtype=dtype, korder=korder, mask="logits", seed=41)
    d = wl.make_inputs(L)
    rng = np.random.Generator(np.random.PCG64(7))
    scale = np.float32(2.0 ** rng.integers(-12, 3, size=d["W"].shape))     # updates from far below an ulp to larger than W
    Ub = wl.to_bits(rng.standard_normal(d["W"].shape, dtype=np.float32) * scale, dtype)
    Wb = d["W"].copy()
    edge = [(0x0001, 0x0001), (0x8000, 0x0000), (0x7BFF if dtype == wl.F16 else 0x7F7F, 0x7BFF if dtype == wl.F16 else 0x7F7F),
            (0x3C00, 0xBC00), (0x03FF, 0x0001)]
    for i, (a, b) in enumerate(edge[:min(len(edge), Wb.size)]):
        Wb.reshape(-1)[i], Ub.reshape(-1)[i] = a, b
    V = oracle.update(Wb, Ub, dtype)
    desc = layer_desc(ss, L)
    W, U, M = dev_bits(Wb, dtype), dev_bits(Ub, dtype), torch.from_numpy(d["M"]).cuda()
    U_before = U.clone()
    packed = ss.ss_mask_update_compress(desc, W, U, M)
    assert np.array_equal(host_bits(W), V)
    assert torch.equal(U.view(torch.int16), U_before.view(torch.int16))
    vals, meta = oracle.compress(V, d["M"])
    assert np.array_equal(packed.cpu().numpy(), dl.tile(vals, meta, cin=cin, kh=kh, kw=kw, dtype=dtype, korder=korder))
    # the same bytes as packing the updated weights from scratch
    assert torch.equal(packed, ss.ss_mask_compress(desc, W, M))


def test_convolution_after_an_update_uses_the_new_weights(ss):
    L = wl.Layer("t", N=2, H=9, W=9, cin=64, cout=96, kh=3, kw=3, stride=1, pad=1, dtype=wl.BF16, act=wl.ACT_RELU,
                 mask="logits", seed=12)
    d = wl.make_inputs(L)
    rng = np.random.Generator(np.random.PCG64(8))
    Ub = wl.to_bits(rng.standard_normal(d["W"].shape, dtype=np.float32) * np.float32(0.05), L.dtype)
    desc = layer_desc(ss, L)
    W, U, M = dev_bits(d["W"], L.dtype), dev_bits(Ub, L.dtype), torch.from_numpy(d["M"]).cuda()
    packed = ss.ss_mask_update_compress(desc, W, U, M)
    y = ss.ss_conv2d_fwd(desc, dev_bits(d["x"], L.dtype), packed, torch.from_numpy(d["bias"]).cuda(), (1, 1), (1, 1), L.act)
    V = oracle.update(d["W"], Ub, L.dtype)
    ref = oracle.conv2d(d["x"], V, d["M"], cin=L.cin, kh=3, kw=3, dtype=L.dtype, bias=d["bias"], pad=(1, 1), act=L.act)
    from helpers import check_close
    check_close(y, ref, "conv after update")
    old = oracle.conv2d(d["x"], d["W"], d["M"], cin=L.cin, kh=3, kw=3, dtype=L.dtype, bias=d["bias"], pad=(1, 1), act=L.act)
    assert np.linalg.norm(ref - old) / np.linalg.norm(old) > 0.05          # the update is visible at this tolerance


def test_update_compress_argument_and_mask_errors(ss):
    L = wl.Layer("t", N=1, H=2, W=2, cin=16, cout=40, kh=1, kw=1, mask="logits", seed=1)
    d = wl.make_inputs(L)
    desc = layer_desc(ss, L)
    W, M = dev_bits(d["W"], L.dtype), torch.from_numpy(d["M"]).cuda()
    with pytest.raises(ss.SSError):
        ss.ss_mask_update_compress(desc, W, W[:10], M)
    Mb = d["M"].copy()
    Mb[3, 4:8] = [1, 1, 1, 0]
    U = torch.zeros_like(W)
    with pytest.raises(ss.SSError) as e:
        ss.ss_mask_update_compress(desc, W, U, torch.from_numpy(Mb).cuda())
    assert e.value.status == ss.SS_ERR_BAD_MASK and e.value.detail == (3, 1)


@pytest.mark.parametrize("K,offset", [(8, 0), (12, 0), (147, 0), (264, 0), (264, 1), (260, 4), (516, 0)])
def test_dense_pack_reads_rows_of_any_alignment(ss, K, offset):
    """Rows of 16-, 8- and 2-byte units, and operands whose address allows less than the row length does; odd step counts."""
    cout = 37
    rng = np.random.Generator(np.random.PCG64(K + offset))
    W = rng.integers(0, 1 << 16, size=cout * K + offset, dtype=np.uint16)
    M = rng.integers(0, 2, size=cout * K + offset, dtype=np.uint8)
    desc = ss.make_desc(cout, K, 1, 1, wl.F16)
    got = ss.ss_dense_pack(desc, dev_bits(W, wl.F16)[offset:], torch.from_numpy(M).cuda()[offset:]).cpu().numpy()
    Wm = np.where(M == 1, W, 0).astype(np.uint16)[offset:].reshape(cout, K)
    assert np.array_equal(got, dl.tile_dense(Wm, cin=K, kh=1, kw=1, dtype=wl.F16, korder=wl.K_CRS))


@pytest.mark.parametrize("mode", ["global", "thread_local", "relaxed"])
def test_packing_calls_that_wait_are_refused_under_capture(ss, mode):
    """A recorded compression could report no mask: refused with nothing recorded, and the capture goes on."""
    L = wl.Layer("t", N=1, H=4, W=4, cin=64, cout=64, kh=1, kw=1, dtype=wl.BF16, mask="logits", seed=3)
    d = wl.make_inputs(L)
    desc = layer_desc(ss, L)
    W, M = dev_bits(d["W"], L.dtype), torch.from_numpy(d["M"]).cuda()
    U, W_before = torch.ones_like(W), W.clone()
    packed = ss.ss_mask_compress(desc, W, M)
    want = packed.clone()
    launch, y = ss.prepare_conv2d(desc, dev_bits(d["x"], L.dtype), packed, None, (1, 1), (0, 0), L.act)
    launch()
    torch.cuda.synchronize()
    eager = host_bits(y).copy()
    # The graph of the mode before lives in a reference cycle (exception -> traceback -> frame).  Collected during the capture, its destructor
    # synchronizes the device, which is refused there, and an exception in a destructor ends the process.
    gc.collect()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, capture_error_mode=mode):
        launch()
        for call in (lambda: ss.ss_mask_compress(desc, W, M, packed=packed), lambda: ss.ss_mask_update_compress(desc, W, U, M, packed=packed),
                     lambda: ss.ss_mask_update_compress(desc, W, U, M, packed=packed, stream=torch.cuda.current_stream())):
            with pytest.raises(ss.SSError) as e:
                call()
            assert e.value.status == ss.SS_ERR_HIP
    for _ in range(3):
        y.zero_()
        g.replay()
        torch.cuda.synchronize()
        assert np.array_equal(host_bits(y), eager)
        assert torch.equal(W, W_before) and torch.equal(packed, want)
    ss.ss_mask_update_compress(desc, W, U, M, packed=packed)                 # and the calls still work afterwards
    assert np.array_equal(host_bits(W), oracle.update(d["W"], host_bits(U), L.dtype))


def test_update_of_a_lazy_clone_leaves_the_original_alone(ss):
    """W is written through an address for writing: a clone that still shares its memory gets memory of its own first."""
    L = wl.Layer("t", N=1, H=2, W=2, cin=64, cout=40, kh=1, kw=1, dtype=wl.BF16, mask="logits", seed=5)
    d = wl.make_inputs(L)
    W, M = dev_bits(d["W"], L.dtype), torch.from_numpy(d["M"]).cuda()
    clone, U = torch._lazy_clone(W), torch.ones_like(W)
    ss.ss_mask_update_compress(layer_desc(ss, L), clone, U, M)
    assert np.array_equal(host_bits(W), d["W"])
    assert np.array_equal(host_bits(clone), oracle.update(d["W"], host_bits(U), L.dtype))


@pytest.mark.parametrize("rows,steps", [(1, 1), (3, 84), (4, 64), (1, 260), (9, 60)])
def test_verdict_of_grids_of_any_size(ss, rows, steps):
    """The verdict comes from the last of the grid's workgroups (one for 32 rows x 4 steps: 1, 63, 64, 65 and 135 of them here; from 64 on they
    count in sixteen groups), covers every one of them, and leaves the counters ready for the next call; what was packed is there for
    another stream as soon as the call returns."""
    cout, K = 32 * rows - 5, 32 * steps - 8
    rng = np.random.Generator(np.random.PCG64(steps))
    W = rng.integers(0, 1 << 16, size=(cout, K), dtype=np.uint16)
    M = wl.mask_from_logits(rng.standard_normal((cout, K // 4, 6)).astype(np.float32)).reshape(cout, K)
    desc = ss.make_desc(cout, K, 1, 1, wl.F16)
    vals, meta = oracle.compress(W, M)
    want = dl.tile(vals, meta, cin=K, kh=1, kw=1, dtype=wl.F16, korder=wl.K_CRS)
    Wd, Md = dev_bits(W, wl.F16), torch.from_numpy(M).cuda()
    other = torch.cuda.Stream()
    out = torch.empty(want.size, dtype=torch.uint8, device="cuda")
    torch.cuda.synchronize()
    for i in range(6):
        out.fill_(0xA5)
        ss.ss_mask_compress(desc, Wd, Md, packed=out)
        with torch.cuda.stream(other):
            got = out.cpu().numpy()
        assert np.array_equal(got, want)
        row, block = (cout - 1, K // 4 - 1) if i % 2 else (0, 0)
        wrong = Md.clone()
        wrong[row, 4 * block:4 * block + 4] = 1
        with pytest.raises(ss.SSError) as e:
            ss.ss_mask_compress(desc, Wd, wrong)
        assert e.value.status == ss.SS_ERR_BAD_MASK and e.value.detail == (row, block)


@pytest.mark.parametrize("dtype", [wl.F16, wl.BF16])
@pytest.mark.parametrize("rows,steps", [(1, 1), (9, 60)])
def test_updated_weights_are_there_for_another_stream(ss, rows, steps, dtype):
    """As soon as the call returns, the weights it moved are there for a copy on another stream, with what was packed from them."""
    cout, K = 32 * rows - 5, 32 * steps - 8
    rng = np.random.Generator(np.random.PCG64(rows))
    W = wl.to_bits(rng.standard_normal((cout, K), dtype=np.float32), dtype)
    U = wl.to_bits(rng.standard_normal((cout, K), dtype=np.float32) * np.float32(0.1), dtype)
    M = wl.mask_from_logits(rng.standard_normal((cout, K // 4, 6)).astype(np.float32)).reshape(cout, K)
    desc, Ud, Md = ss.make_desc(cout, K, 1, 1, dtype), dev_bits(U, dtype), torch.from_numpy(M).cuda()
    other, out = torch.cuda.Stream(), torch.empty(dl.tile(*oracle.compress(W, M), cin=K, kh=1, kw=1, dtype=dtype, korder=wl.K_CRS).size,
                                                  dtype=torch.uint8, device="cuda")
    Wd = dev_bits(W, dtype)
    torch.cuda.synchronize()
    for _ in range(4):
        W = oracle.update(W, U, dtype)
        ss.ss_mask_update_compress(desc, Wd, Ud, Md, packed=out)
        with torch.cuda.stream(other):
            moved, packed = Wd.view(torch.int16).cpu().numpy().view(np.uint16), out.cpu().numpy()
        assert np.array_equal(moved, W)
        assert np.array_equal(packed, dl.tile(*oracle.compress(W, M), cin=K, kh=1, kw=1, dtype=dtype, korder=wl.K_CRS))


def test_a_call_that_reports_an_earlier_error_has_waited_for_its_kernel(ss):
    """The runtime keeps an error of the thread until it is asked for it; a packing call that finds one reports it, but not before
    its kernel is done: what the call waits with is free again (a device has sixteen sets of counters), and so are its buffers."""
    L = wl.Layer("t", N=1, H=4, W=4, cin=64, cout=64, kh=1, kw=1, dtype=wl.F16, mask="logits", seed=5)
    d, desc = wl.make_inputs(L), layer_desc(ss, L)
    W, M = dev_bits(d["W"], L.dtype), torch.from_numpy(d["M"]).cuda()
    want = ss.ss_mask_compress(desc, W, M)
    packed = torch.zeros_like(want)
    with open("/proc/self/maps") as maps:
        hip = ctypes.CDLL(next(line.split()[-1] for line in maps if "libamdhip64" in line))
    stream, other, want_host = torch.cuda.current_stream(), torch.cuda.Stream(), want.cpu().numpy()
    torch.cuda.synchronize()
    for _ in range(20):
        torch.cuda._sleep(2_000_000)
        assert hip.hipSetDevice(1 << 20) != 0
        status = binding._lib.ss_mask_compress(ctypes.byref(desc), W.data_ptr(), M.data_ptr(), packed.data_ptr(), None, stream.cuda_stream)
        if status == ss.SS_OK:
            pytest.skip("this runtime forgets an error with the next call that succeeds")
        assert status == ss.SS_ERR_HIP
        with torch.cuda.stream(other):                    # (does not wait for the call's stream)
            assert np.array_equal(packed.cpu().numpy(), want_host)
        packed.zero_()
    assert torch.equal(ss.ss_mask_compress(desc, W, M), want)
