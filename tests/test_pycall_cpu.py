"""The marshalling module takes what ctypes takes for the same declarations, and refuses what ctypes refuses.
(No GPU: every call ends in the library's own argument checks.)"""
import ctypes as C

import numpy as np
import pytest

from tests.test_abi_cpu import A, _shape, fb


def _status(fn, *a):
    try:
        fn(*a)
    except fb.FasaError as e:
        return e.status
    return 0


@pytest.mark.parametrize("as_int", [int, np.int64, np.uint64, np.int32], ids=lambda t: t.__name__)
def test_sizes_and_ranges_are_any_integer(as_int):
    s = _shape()
    need = fb.fasa_workspace_bytes(s)
    for size in (as_int(0), as_int(need - 1)):
        assert _status(fb.fasa_topk, s, A, A, A, size, 0) == fb.FASA_EWORKSPACE
    # large enough a size gets past its check: to the pointer's
    assert _status(fb.fasa_topk, s, A, A, None, as_int(need), 0) == fb.FASA_EINVAL
    assert _status(fb.fasa_pack_kcache, s, A, A, A, as_int(7), as_int(7), 0) == 0          # empty range
    assert _status(fb.fasa_pack_kcache, s, A, A, A, as_int(9), as_int(7), 0) == fb.FASA_EINVAL
    assert _status(fb.fasa_offload_decode_step, s, A, A, A, A, A, None, None, A, A, A, A, as_int(need), A, as_int(16), 0) == fb.FASA_EWORKSPACE
    assert _status(fb.fasa_contextual_agreement, s, A, A, as_int(64), A, A, as_int(16), 0) == fb.FASA_EWORKSPACE


def test_integers_are_reduced_as_by_ctypes():
    s = _shape()
    for n0, n1 in ((-1, 5), ((1 << 32) + 9, 7), ((1 << 65) + 9, 7), (True, 0)):       # (all of them refused)
        want = fb.lib.fasa_pack_kcache(C.byref(s), A, A, A, n0, n1, None)
        assert want == fb.FASA_EINVAL and _status(fb.fasa_pack_kcache, s, A, A, A, n0, n1, 0) == want
    assert _status(fb.fasa_topk, s, A, A, None, -1, 0) == fb.FASA_EINVAL
    for bad in (5.0, "5", None, np.float64(5)):
        with pytest.raises(TypeError):
            fb.fasa_topk(s, A, A, A, bad, 0)


def test_structures_are_checked_by_type():
    """A call takes the binding's own structures (and what derives from them), nothing that merely has as many bytes."""
    class Shape(fb.FasaShape):
        pass

    s, pg = _shape(), fb.FasaPaging(A, 64, 16, 100, 0)
    own = Shape.from_buffer_copy(s)
    assert _status(fb.fasa_topk, own, A, A, A, 0, 0) == fb.FASA_EWORKSPACE
    step = lambda shape, paging: fb.fasa_decode_step_paged(shape, paging, A, A, A, A, A, None, None, None, None, A, A, A, A, 0, 0)
    assert _status(step, own, pg) == fb.FASA_EWORKSPACE
    for other in (bytearray(bytes(s)), bytes(s), np.zeros(64, np.uint8), None, 0, A):
        with pytest.raises(TypeError):
            fb.fasa_topk(other, A, A, A, 0, 0)
        with pytest.raises(TypeError):
            step(s, other)
    for other in (pg, C.pointer(s), (fb.FasaShape * 1)(s), C.create_string_buffer(bytes(s))):
        with pytest.raises(C.ArgumentError):
            fb.lib.fasa_topk(C.byref(other), A, A, A, 0, None)
        with pytest.raises(C.ArgumentError):
            fb.fasa_topk(other, A, A, A, 0, 0)
    with pytest.raises(C.ArgumentError):
        step(s, s)


def test_the_first_refused_argument_is_reported():
    """Also where a later argument goes through a path of its own (an array's address, a bad size, a bad stream)."""
    with pytest.raises(TypeError, match="ctypes instance"):
        fb.fasa_topk("no shape", np.zeros(4, np.float32), object(), A, "no size", "no stream")
    with pytest.raises(TypeError, match="address"):
        fb.fasa_topk(_shape(), object(), np.zeros(4, np.int32), A, "no size", "no stream")


def _import_error(tmp_path, module):
    """The message of importing a copy of the package whose marshalling module is the given bytes (None: not there)."""
    import os
    import subprocess
    import sys
    pkg = tmp_path / "paper_2602_03152_amd"
    pkg.mkdir(parents=True)
    src = os.path.dirname(fb.__file__)
    for name in ("__init__.py", "binding.py"):
        (pkg / name).write_bytes(open(os.path.join(src, name), "rb").read())
    os.symlink(fb._LIB_PATH, pkg / "libfasa.so")
    if module is not None:
        (pkg / os.path.basename(fb._pycall.__file__)).write_bytes(module)
    p = subprocess.run([sys.executable, "-c", "import paper_2602_03152_amd.binding"], cwd=tmp_path, text=True,
                       env={k: v for k, v in os.environ.items() if k != "FASA_LIB"}, stderr=subprocess.PIPE, timeout=100)
    assert p.returncode != 0
    return p.stderr.strip().splitlines()[-1]


def test_a_module_that_is_missing_is_told_from_one_that_does_not_load(tmp_path):
    assert "not built" in _import_error(tmp_path / "a", None)
    msg = _import_error(tmp_path / "b", b"not a shared object")
    assert "not built" not in msg and "cannot be loaded" in msg
