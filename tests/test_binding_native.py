"""The native call path of the binding: it takes plain device tensors and leaves everything else to the checks in Python."""
import ctypes
import types

import pytest
import torch

import paper_1803_09926_amd as dw


class Sub(torch.Tensor):
    pass


CALLS = {"fwd": "xwy", "bwd_data": "ywx", "bwd_filter": "xyds", "bwd_filter_noalloc": "xyd", "bwd": "xywxds",
         "gconv_fwd": "xwy", "gconv_bwd_data": "ywx", "gconv_bwd_filter": "xyds"}


def _operands(name, device):
    group = name.startswith("gconv")
    d = dw.group_desc(2, 8, 9, 9, groups=2) if group else dw.desc(2, 8, 9, 9)
    t = {"x": torch.ones(2, 8, 9, 9), "y": torch.ones(2, 8, 9, 9), "w": torch.ones((8, 4, 3, 3) if group else (8, 3, 3)),
         "d": torch.zeros((8, 4, 3, 3) if group else (8, 3, 3)), "s": torch.zeros(1 << 16, dtype=torch.uint8)}
    return d, [t[k].clone().to(device) for k in CALLS[name]]


@pytest.mark.parametrize("name", CALLS)
def test_host_tensors_and_other_descriptors_are_left_to_python(name):
    d, t = _operands(name, "cpu")
    native = dw._native or dw._bind_native()
    assert getattr(native, name)(d, *t, None) is None
    assert getattr(native, name)(object(), *t, None) is None
    with pytest.raises(ValueError, match="device tensor"):
        getattr(dw, name)(d, *t)
    with pytest.raises(TypeError):
        getattr(native, name)(d)
    bad = dw.group_desc(2, 8, 9, 9, groups=0) if name.startswith("gconv") else dw.desc(2, 8, 1, 1, 5, 1, 0)
    with pytest.raises(dw.DwconvError):
        getattr(dw, name)(bad, *t)


@pytest.mark.gpu
@pytest.mark.parametrize("name", CALLS)
def test_every_call_by_both_ways(gpu_lib, name):
    d, t = _operands(name, "cuda")
    native, side = dw._native or dw._bind_native(), torch.cuda.Stream()
    getattr(dw, name)(d, *t)
    want = [v.clone() for v in t]

    def agrees(form, stream=None):
        d, t = _operands(name, "cuda")
        torch.cuda.synchronize()
        getattr(dw, name)(d, *[form(v) for v in t], stream=stream)
        torch.cuda.synchronize()
        for k, a, b in zip(CALLS[name], t, want):
            assert k == "s" or torch.equal(a, b)
    agrees(lambda v: v, side)
    agrees(lambda v: torch.nn.Parameter(v, requires_grad=False))
    agrees(lambda v: v.as_subclass(Sub))                                  # a subclass: by the checks in Python
    assert getattr(native, name)(d, *[v.as_subclass(Sub) for v in t], None) is None
    for i, k in enumerate(CALLS[name]):
        if k == "s":
            continue
        for wrong in (t[i].double(), t[i].flatten()[1:], t[i].cpu(), torch.stack([t[i], t[i]], -1)[..., 0]):
            args = t[:i] + [wrong] + t[i + 1:]
            assert getattr(native, name)(d, *args, None) is None
            with pytest.raises(ValueError):
                getattr(dw, name)(d, *args)
    if "s" in CALLS[name]:
        with pytest.raises(dw.DwconvError):
            getattr(dw, name)(d, *t[:-1], t[-1][:4])


@pytest.mark.gpu
@pytest.mark.parametrize("name", CALLS)
def test_stream_handles_of_every_form_that_a_pointer_takes(gpu_lib, name):
    """A handle that is no number is left to the foreign call, which takes None (the null stream) and c_void_p as well."""
    d, t = _operands(name, "cuda")
    native, side = dw._native or dw._bind_native(), torch.cuda.Stream()
    getattr(dw, name)(d, *t)
    torch.cuda.synchronize()
    for handle, plain in ((side.cuda_stream, True), (ctypes.c_void_p(side.cuda_stream), False), (0, True), (None, False), (ctypes.c_void_p(None), False)):
        stream = types.SimpleNamespace(cuda_stream=handle)
        _, got = _operands(name, "cuda")
        torch.cuda.synchronize()
        assert (getattr(native, name)(d, *got, stream) is None) != plain
        getattr(dw, name)(d, *got, stream=stream)
        torch.cuda.synchronize()
        for k, a, b in zip(CALLS[name], got, t):
            assert k == "s" or torch.equal(a, b)
    with pytest.raises(ctypes.ArgumentError):
        getattr(dw, name)(d, *t, stream=types.SimpleNamespace(cuda_stream=1.5))
    with pytest.raises(AttributeError):
        getattr(dw, name)(d, *t, stream=object())


@pytest.mark.gpu
def test_wrapped_tensors_raise(gpu_lib):
    d, t = _operands("fwd", "cuda")
    with pytest.raises(Exception):
        torch.vmap(lambda v: dw.fwd(d, v, t[1], t[2]))(torch.stack([t[0], t[0]]))
    with pytest.raises(Exception):
        torch.func.jvp(lambda v: dw.fwd(d, v, t[1], t[2]), (t[0],), (t[0],))
