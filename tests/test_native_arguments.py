"""CPU tests of the argument marshalling in csrc/sc_python.cpp: shapes, types and devices that a call refuses
before it looks at a device pointer, so no GPU is needed; and (one needs device tensors, but launches
nothing) the interpreter lock around the library's calls."""
import ctypes

import pytest
import torch

from paper_2402_07710_amd import binding as sc

F16 = torch.float16


def feat(*shape, dtype=F16):
    return torch.zeros(shape, dtype=dtype)


WEIGHT = feat(27, 32, 64)


@pytest.mark.parametrize("feat_in,feat_out,weight,what", [
    (feat(10, 32, 1), feat(10, 64), WEIGHT, "feat_in must be"),
    (feat(10, 32, 5), feat(10, 64), WEIGHT, "feat_in must be"),
    (feat(320), feat(10, 64), WEIGHT, "feat_in must be"),
    (feat(10, 32), feat(10, 64, 5), WEIGHT, "feat_out must be"),
    (feat(10, 32), feat(640), WEIGHT, "feat_out must be"),
    (feat(10, 16), feat(10, 64), WEIGHT, "weight must be"),
    (feat(10, 32), feat(10, 32), WEIGHT, "weight must be"),
    (feat(10, 32), feat(10, 64), WEIGHT[:8], "weight must be"),
    (feat(10, 32), feat(10, 64), WEIGHT.flatten(), "weight must be"),
    (feat(10, 32), feat(10, 64), WEIGHT.to(torch.bfloat16), "weight must be"),
    (feat(10, 32), feat(10, 64), WEIGHT, "device tensor expected"),          # everything fits but the device
])
def test_conv_fwd_refuses(feat_in, feat_out, weight, what):
    with pytest.raises(ValueError, match=what):
        sc.sc_conv_fwd(feat_in, weight, feat_out, feat(1), feat(1), 3, 1, "subm", None, 0)


@pytest.mark.parametrize("feat_in,feat_out,what", [
    (feat(10, 32, 1), feat(10, 64), "feat_in must be"),
    (feat(320), feat(10, 64), "feat_in must be"),
    (feat(10, 32), feat(10, 64, 5), "feat_out must be"),
    (feat(10, 32), feat(10, 32), "feat_out must have C_out columns"),
    (feat(10, 32), feat(10, 64), "device tensor expected"),
])
def test_conv_fwd_packed_refuses(feat_in, feat_out, what):
    with pytest.raises(ValueError, match=what):
        sc.sc_conv_fwd_packed(feat_in, feat(1), 64, feat_out, feat(1), feat(1), 3, 1, "subm", 0)


@pytest.mark.parametrize("coarse,fine", [(feat(4, 32, 5), feat(10, 64)), (feat(128), feat(10, 64)), (feat(4, 16), feat(10, 64)),
                                         (feat(4, 32), feat(10, 64, 5)), (feat(4, 32), feat(9, 64)), (feat(4, 32), feat(10, 32)),
                                         (feat(4, 32, dtype=torch.float32), feat(10, 64))])
def test_conv_up_fwd_refuses(coarse, fine):
    with pytest.raises(sc.ScError) as e:
        sc.sc_conv_up_fwd(coarse, 10, feat(8, 32, 64), fine, feat(1), feat(1), 2, 0)
    assert e.value.code == sc.SC_EINVAL


def test_other_arguments():
    with pytest.raises(TypeError, match="tensor expected"):
        sc.sc_conv_fwd([[1.0]], WEIGHT, feat(10, 64), feat(1), feat(1), 3, 1, "subm", None, 0)
    with pytest.raises(TypeError, match="dims must be"):
        sc.sc_grid_build(feat(4, 4), feat(1), (1, 2, 3), 1, feat(1), 0)
    with pytest.raises(OverflowError):
        sc.sc_grid_build(feat(4, 4), feat(1), (1, 2, 3, 1 << 40), 1, feat(1), 0)
    with pytest.raises(ValueError, match="device tensor expected"):
        sc.sc_hash_build(torch.zeros((4, 4), dtype=torch.int32), feat(1), feat(1), 0)


@pytest.fixture
def lock_held():
    """The module with every library function replaced by CPython's PyGILState_Check: a call returns 1
    if the library would run with the interpreter lock held, else 0."""
    lib = sc.load()
    check = ctypes.cast(ctypes.pythonapi.PyGILState_Check, ctypes.c_void_p).value
    sc._native.bind(*[check] * len(sc._NATIVE_CALLS))
    yield sc._native
    sc._native.bind(*(ctypes.cast(getattr(lib, name), ctypes.c_void_p).value for name in sc._NATIVE_CALLS))


def test_a_call_releases_the_interpreter_lock(lock_held):
    assert lock_held.kmap_transpose(None, 10, 2, 2, None, None, 0) == 0


@pytest.mark.gpu
def test_every_call_releases_the_interpreter_lock(lock_held):
    def dev(*shape, dtype=F16):
        return torch.zeros(shape, dtype=dtype, device="cuda:0")
    xyz, buf, dims = dev(4, 4, dtype=torch.int32), dev(1), (1, 8, 8, 8)
    calls = dict(hash_build=(xyz, buf, buf, None), hash_rebuild=(xyz, buf, 1, buf, None),
                 kmap_build=(xyz, buf, 3, 1, 0, None, buf, buf, buf, None), kmap_build_noalloc=(xyz, buf, 3, 1, 0, None, buf, buf, None),
                 kmap_transpose=(buf, 4, 2, 2, buf, buf, None), grid_build=(xyz, buf, dims, 1, buf, None),
                 kmap_build_grid=(xyz, buf, dims, 1, 3, buf, buf, None),
                 conv_fwd=(dev(4, 32), None, dev(27, 32, 32), dev(4, 32), buf, buf, 3, 1, 0, buf, None),
                 conv_fwd_packed=(dev(4, 32), None, buf, 32, dev(4, 32), buf, buf, 3, 1, 0, None),
                 conv_up_fwd=(dev(4, 64), 4, dev(8, 64, 32), dev(4, 32), buf, buf, 2, None),
                 conv_fwd_grid=(dev(4, 32), xyz, buf, dims, 1, dev(27, 32, 32), dev(4, 32), 3, buf, None))
    assert sorted("sc_" + name for name in calls) == sorted(sc._NATIVE_CALLS)
    for name, args in calls.items():
        assert getattr(lock_held, name)(*args) == 0, name
