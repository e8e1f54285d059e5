"""Calls from several Python threads: a call that blocks gives the interpreter to the others, and concurrent calls on streams of
their own do not disturb each other."""
import threading
import time

import numpy as np
import pytest
import torch

import oracle
from oracle import device_layout as dl
from paper_2411_00288_amd import workloads as wl
from helpers import check_close, dev_bits, layer_desc, oracle_ref

pytestmark = pytest.mark.gpu


def _layer(seed=0, **kw):
    args = dict(N=1, H=8, W=8, cin=64, cout=64, kh=1, kw=1, dtype=wl.BF16, mask="logits", seed=seed)
    return wl.Layer("t", **dict(args, **kw))


def _sleep(seconds):
    """Keeps the GPU busy for about this long (a kernel that counts clocks)."""
    torch.cuda._sleep(100_000)
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    torch.cuda._sleep(10_000_000)
    torch.cuda.synchronize()
    torch.cuda._sleep(int(10_000_000 * seconds / (time.perf_counter() - t0)))


class _Ticker:
    """A second thread that wants to run every millisecond; `worst` is the longest it had to wait."""
    def __enter__(self):
        self.stop, self.worst = threading.Event(), 0.0
        def run():
            last = time.perf_counter()
            while not self.stop.is_set():
                time.sleep(0.001)
                now = time.perf_counter()
                self.worst, last = max(self.worst, now - last), now
        self.thread = threading.Thread(target=run)
        self.thread.start()
        return self
    def __exit__(self, *exc):
        self.stop.set()
        self.thread.join()


@pytest.mark.parametrize("how", ["call", "prepared"])
def test_a_launch_into_a_full_queue_lets_other_threads_run(ss, how):
    L = _layer()
    d = wl.make_inputs(L)
    desc, x = layer_desc(ss, L), dev_bits(d["x"], L.dtype)
    w = ss.ss_mask_compress(desc, dev_bits(d["W"], L.dtype), torch.from_numpy(d["M"]).cuda())
    launch, y = ss.prepare_conv2d(desc, x, w)
    call = launch if how == "prepared" else lambda: ss.ss_conv2d_fwd(desc, x, w, y=y)
    call()
    torch.cuda.synchronize()
    _sleep(0.3)
    longest = 0.0
    with _Ticker() as other:
        for _ in range(20000):                       # more than the queue takes (it was full after about 2700)
            t0 = time.perf_counter()
            call()
            longest = max(longest, time.perf_counter() - t0)
    torch.cuda.synchronize()
    if longest < 0.1:
        pytest.skip("the queue took every launch")
    assert other.worst < longest / 2                 # (the lock held: as long as the launch itself)


def test_a_packing_call_that_waits_lets_other_threads_run_and_sleeps(ss):
    L = _layer(seed=1)
    d = wl.make_inputs(L)
    desc, W, M = layer_desc(ss, L), dev_bits(d["W"], L.dtype), torch.from_numpy(d["M"]).cuda()
    want = ss.ss_mask_compress(desc, W, M)
    _sleep(0.3)
    wall, cpu = time.perf_counter(), time.thread_time()
    with _Ticker() as other:
        got = ss.ss_mask_compress(desc, W, M)
    wall, cpu = time.perf_counter() - wall, time.thread_time() - cpu
    assert torch.equal(got, want)
    if wall < 0.1:
        pytest.skip("the GPU was not kept busy")
    assert other.worst < wall / 2
    assert cpu < wall / 2                            # (polling throughout: all of it)


def test_concurrent_calls_on_their_own_streams(ss):
    """Packing (pinned words and events handed out per call) and a split reduction (a workspace per stream) from eight threads."""
    L = _layer(N=3, H=20, W=20, cin=512, cout=512, kh=3, kw=3, pad=1, seed=2)
    d = wl.make_inputs(L)
    ref = oracle_ref(L, d)
    desc = layer_desc(ss, L)
    assert ss.ss_conv2d_workspace_bytes(desc, L.N, L.H, L.W, (1, 1), (1, 1)) > 0
    vals, meta = oracle.compress(d["W"], d["M"])
    bytes_ = torch.from_numpy(dl.tile(vals, meta, cin=L.cin, kh=3, kw=3, dtype=L.dtype, korder=L.korder)).cuda()
    x, W, M = dev_bits(d["x"], L.dtype), dev_bits(d["W"], L.dtype), torch.from_numpy(d["M"]).cuda()
    bad = M.clone()
    bad[7, 20:24] = 1
    bias = torch.from_numpy(d["bias"]).cuda()
    torch.cuda.synchronize()
    results, errors = [], []
    def work(i):
        try:
            stream = torch.cuda.Stream()
            with torch.cuda.stream(stream):
                for _ in range(5):
                    packed = ss.ss_mask_compress(desc, W, M)
                    if i % 2:                        # other calls' findings do not leak into this one
                        with pytest.raises(ss.SSError) as e:
                            ss.ss_mask_compress(desc, W, bad)
                        assert e.value.detail == (7, 5)
                    y = ss.ss_conv2d_fwd(desc, x, packed, bias, (1, 1), (1, 1), L.act)
                stream.synchronize()
                results.append((packed, y))
        except BaseException as e:                   # noqa: BLE001  (reported by the main thread)
            errors.append(e)
    threads = [threading.Thread(target=work, args=(i,)) for i in range(8)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not errors, errors
    assert len(results) == 8
    for packed, y in results:
        assert torch.equal(packed, bytes_)
        check_close(y, ref, "concurrent call")
        assert torch.equal(y, results[0][1])         # sums in a fixed order: the same bits from every thread


def test_more_packing_calls_at_once_than_there_are_counters(ss):
    """Sixteen calls in flight wait for their last workgroup, further ones for an event: 24 threads, each behind work of its own."""
    L = _layer(cin=64, cout=96, kh=3, kw=3, pad=1, seed=4)
    d = wl.make_inputs(L)
    desc, W, M = layer_desc(ss, L), dev_bits(d["W"], L.dtype), torch.from_numpy(d["M"]).cuda()
    want = ss.ss_mask_compress(desc, W, M)
    wrong = M.clone()
    wrong[11, 8:12] = 0
    torch.cuda.synchronize()
    results, errors, start = [], [], threading.Barrier(24)

    def work(i):
        try:
            with torch.cuda.stream(torch.cuda.Stream()):
                start.wait()
                for _ in range(3):
                    torch.cuda._sleep(2_000_000)             # about a millisecond
                    results.append(ss.ss_mask_compress(desc, W, M))
                    with pytest.raises(ss.SSError) as e:
                        ss.ss_mask_compress(desc, W, wrong)
                    assert e.value.detail == (11, 2)
        except BaseException as e:                   # noqa: BLE001  (reported by the main thread)
            errors.append(e)
    threads = [threading.Thread(target=work, args=(i,)) for i in range(24)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not errors, errors
    assert len(results) == 72 and all(torch.equal(r, want) for r in results)
