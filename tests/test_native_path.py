"""The compiled call path of the binding (csrc/ss_python.cpp) on the CPU: it declines whatever is not the plain good case, and the
checked path then raises what it always raised.  Device tensors that need no device are FakeTensors."""
import warnings

import pytest
import torch
from torch._subclasses.fake_tensor import FakeTensorMode

import paper_2411_00288_amd as ss
from paper_2411_00288_amd import binding

ONE = (1, 1)


@pytest.fixture
def fake():
    """Operands of small calls as device tensors without memory (names as in the calls below)."""
    with warnings.catch_warnings(), FakeTensorMode(allow_non_fake_inputs=True):
        warnings.simplefilter("ignore")
        def dev(*shape, dtype=torch.float16):
            return torch.empty(shape, dtype=dtype, device="cuda")
        d, d2, d8 = ss.make_desc(64, 64, 3, 3), ss.make_desc(64, 64, 1, 1), ss.make_desc(64, 64, 3, 3, ss.SS_I8)
        def packed(desc):
            return dev(ss.ss_packed_bytes(desc), dtype=torch.uint8)
        yield {"d": d, "d2": d2, "d8": d8, "x": dev(1, 8, 8, 64), "x8": dev(1, 8, 8, 64, dtype=torch.int8), "w": packed(d),
               "w2": packed(d2), "w8": packed(d8), "dw": dev(7, 7, 64), "dev": dev}


CALLS = {      # one operand of the call comes from torch.func.vmap
    "bias": lambda f, t: ss.ss_conv2d_fwd(f["d"], f["x"], f["w"], t, ONE, ONE),
    "residual": lambda f, t: ss.ss_conv2d_res_fwd(f["d"], f["x"], f["w"], None, t, ONE, ONE),
    "scale": lambda f, t: ss.ss_conv2d_q8_fwd(f["d8"], f["x8"], f["w8"], t, None, ONE, ONE),
    "fused bias": lambda f, t: ss.ss_conv2d_pw_fused_fwd(f["d"], f["x"], f["w"], t, ONE, ONE, 0, f["d2"], f["w2"]),
    "fused residual": lambda f, t: ss.ss_conv2d_pw_fused_fwd(f["d"], f["x"], f["w"], None, ONE, ONE, 0, f["d2"], f["w2"], None, t),
    "depthwise bias": lambda f, t: ss.ss_dwconv2d_fwd(f["x"], f["dw"], t, (3, 3)),
    "input": lambda f, t: ss.ss_conv2d_fwd(f["d"], t, f["w"], None, ONE, ONE),
    "pooling input": lambda f, t: ss.ss_maxpool2d(t),
}


@pytest.mark.parametrize("which", CALLS)
def test_tensors_without_storage_raise_as_the_checked_path_does(fake, which):
    t = fake["dev"](3, 64, dtype=torch.float32) if which.endswith(("bias", "scale")) else fake["dev"](3, 1, 8, 8, 64)
    with pytest.raises(RuntimeError, match="storage"):
        torch.func.vmap(lambda v: CALLS[which](fake, v))(t)


@pytest.mark.parametrize("which", ["W", "U", "M"])
def test_packing_tensors_without_storage_raise_as_the_checked_path_does(fake, which):
    d = fake["d2"]
    t = {k: fake["dev"](64, 64, dtype=torch.uint8 if k == "M" else torch.float16) for k in "WUM"}
    many = fake["dev"](3, 64, 64, dtype=t[which].dtype)
    with pytest.raises(RuntimeError, match="storage"):
        torch.func.vmap(lambda v: ss.ss_mask_update_compress(d, *[v if k == which else t[k] for k in "WUM"]))(many)


def test_compiled_path_declines_and_the_checked_path_gives_the_reason(fake):
    f, nat = fake, binding._native
    host = torch.zeros(1, 8, 8, 64, dtype=torch.float16, device="cpu")
    cases = [                                     # (x, weights, stride, part of the message)
        (host, f["w"], ONE, "device memory"),
        (f["x"][..., :32], f["w"], ONE, "cin channels"),
        (f["x"].transpose(1, 2), f["w"], ONE, "contiguous"),
        (f["x"], f["w"][:-1], ONE, "weight buffer"),
        (f["x"].float(), f["w"], ONE, "dtype"),
        (f["x"], f["w"], (0, 1), "stride"),
    ]
    for x, w, stride, why in cases:
        assert nat.conv(0, f["d"], x, w, None, None, None, stride, ONE, 0, None, None) is None
        with pytest.raises(ss.SSError, match=why) as e:
            ss.ss_conv2d_fwd(f["d"], x, w, None, stride, ONE)
        assert e.value.status == ss.SS_ERR_INVALID_ARG
    assert nat.conv(0, f["d"], f["x"]) is None and nat.pack(0) is None and nat.maxpool() is None      # wrong argument counts
    assert nat.conv(0, b"short", f["x"], f["w"], None, None, None, ONE, ONE, 0, None, None) is None
    assert nat.conv(0, f["d"], f["x"], f["w"], None, None, None, [1, 1], ONE, 0, None, None) is None  # a list as stride


FAILS = {
    "conv": lambda t: ss.ss_conv2d_fwd(t, t, t), "conv residual": lambda t: ss.ss_conv2d_res_fwd(t, t, t, None, t),
    "dense": lambda t: ss.ss_conv2d_dense_fwd(t, t, t), "dense residual": lambda t: ss.ss_conv2d_dense_res_fwd(t, t, t, None, t),
    "q8": lambda t: ss.ss_conv2d_q8_fwd(t, t, t), "q8 dense": lambda t: ss.ss_conv2d_q8_dense_fwd(t, t, t),
    "fused": lambda t: ss.ss_conv2d_pw_fused_fwd(t, t, t, None, ONE, ONE, 0, t, t),
    "fused dense": lambda t: ss.ss_conv2d_pw_fused_dense_fwd(t, t, t, None, ONE, ONE, 0, t, t),
    "pool": lambda t: ss.ss_maxpool2d(t), "depthwise": lambda t: ss.ss_dwconv2d_fwd(t, t),
    "compress": lambda t: ss.ss_mask_compress(t, t, t), "update": lambda t: ss.ss_mask_update_compress(t, t, t, t),
    "dense pack": lambda t: ss.ss_dense_pack(t, t, t),
}


@pytest.mark.parametrize("which", FAILS)
@pytest.mark.parametrize("answer", [(ss.SS_ERR_HIP, -1, -1), (ss.SS_ERR_BAD_MASK, 3, 5)])
def test_a_call_that_failed_after_its_launch_is_not_made_again(monkeypatch, which, answer):
    """Neither through ctypes nor at all: an update that ran twice would have moved the weights twice."""
    made = []
    class Native:
        def __getattr__(self, name):
            return lambda *a: made.append(name) or answer
    class Library:
        def __getattr__(self, name):
            return made.append(name)
        def ss_status_string(self, st):
            return b"status"
    monkeypatch.setattr(binding, "_native", Native())
    monkeypatch.setattr(binding, "_lib", Library())
    with pytest.raises(ss.SSError) as e:
        FAILS[which](object())
    assert (e.value.status, e.value.detail) == (answer[0], (3, 5) if answer[0] == ss.SS_ERR_BAD_MASK else None)
    assert len(made) == 1
