"""The Python binding's native marshalling against ctypes: the same status, or the same exception, for every kind of argument.  Calls that launch
nothing (empty problems, arguments that the entry points refuse)."""
import inspect

import numpy as np
import pytest

import paper_2603_06731_amd as pbk
from paper_2603_06731_amd import binding

pytestmark = pytest.mark.skipif(binding._marshal is None, reason="built without Python's headers")


class Buffer:
    def __init__(self, address=4096):
        self.address = address

    def data_ptr(self):
        return self.address


class Stream:
    cuda_stream = 0


class Broken:
    def data_ptr(self):
        raise RuntimeError("no storage")


X = Buffer()
ENTRIES = [n for n in pbk.EXPORTED_SYMBOLS if hasattr(binding, "_" + n)]


def arguments(name):
    """One valid value per parameter: an empty problem."""
    values = []
    for p in inspect.signature(getattr(pbk, name)).parameters:
        if p in ("A", "B", "C", "x", "w", "y", "Q", "K", "V", "O", "bias", "R", "r", "scale", "mean", "var", "gamma", "beta") and not (
                p == "K" and "matmul" in name) and not (p == "beta" and "residual" in name):
            values.append(X)
        elif p in ("mul", "add"):
            values.append(None)
        elif p == "stream":
            values.append(Stream())
        elif p in ("alpha", "mid_scale", "eps", "out_scale") or p == "beta":
            values.append(0.5)
        elif p in ("M", "batch") or (p == "N" and "conv" in name):
            values.append(0)
        elif p in ("in_dtype", "out_dtype", "dtype"):
            values.append(5 if "int8" in name else 1)
        elif p in ("epi", "trans_b", "relu") or p.startswith(("pad", "out_pad")):
            values.append(0)
        else:
            values.append(8 if not p.startswith(("stride_h", "stride_w", "dil", "KH", "KW")) else 1)
    return values


# the sizes any of which at zero makes the problem empty
SIZES = {n: [i for i, p in enumerate(inspect.signature(getattr(pbk, n)).parameters) if p in ("M", "batch") or (p == "N" and "conv" in n)] for n in ENTRIES}


def outcome(name, args, monkeypatch, native):
    if not native:
        monkeypatch.setattr(binding, "_" + name, lambda *a: None)
    try:
        return getattr(pbk, name)(*args)
    except Exception as e:
        return type(e), str(e)
    finally:
        monkeypatch.undo()


def test_every_entry_point_is_bound():
    binding.lib()
    assert len(ENTRIES) == 13
    for name in ENTRIES:
        args = arguments(name)
        assert getattr(binding._marshal, name)(*args) == getattr(pbk, name)(*args) == 0, name
        assert getattr(binding._marshal, name)(*args[:-1]) is None       # another number of arguments: not judged here


@pytest.mark.parametrize("name", ENTRIES)
@pytest.mark.parametrize("value", [None, 0, 1, -1, True, 1 << 31, -(1 << 31) - 1, 1 << 63, 1 << 64, (1 << 64) + 7, -(1 << 70), 0.5, 1e300, float("nan"),
                                   "8", b"8", np.int64(8), np.float32(0.5), Buffer(0), Buffer(1 << 63), Buffer(-1), Buffer("8"), Broken(), Stream(), object()])
def test_every_argument(name, value, monkeypatch):
    binding.lib()
    base = arguments(name)
    for i in range(len(base)):
        args = base[:i] + [value] + base[i + 1:]
        if i > 0 and 0 not in (args[j] for j in SIZES[name]):
            args[0] = None                                  # no longer an empty problem: refused for a missing operand, so that nothing is ever launched
        got, want = outcome(name, args, monkeypatch, True), outcome(name, args, monkeypatch, False)
        if isinstance(want, tuple) and "object at 0x" in want[1]:
            got, want = got[0], want[0]
        assert got == want, (name, list(inspect.signature(getattr(pbk, name)).parameters)[i], value)


def test_keywords_and_missing_arguments(monkeypatch):
    args = arguments("pbk_matmul")
    names = list(inspect.signature(pbk.pbk_matmul).parameters)
    assert pbk.pbk_matmul(**dict(zip(names, args))) == 0
    assert pbk.pbk_matmul(*args[:-1]) == 0
    with pytest.raises(TypeError):
        pbk.pbk_matmul(*args[:-2])


@pytest.mark.parametrize("error", [KeyboardInterrupt, MemoryError, RuntimeError, AttributeError, TypeError])
def test_an_error_of_the_callers_own(error):
    """What a data_ptr() or cuda_stream raises reaches the caller, and the method does not run once more behind its back (AttributeError and TypeError
    are also what an object without one gives: ctypes judges them)."""
    class Once:
        calls = 0

        def data_ptr(self):
            self.calls += 1
            if self.calls == 1:
                raise error("once")
            return 4096

        cuda_stream = property(data_ptr)

    for at in (0, -1):
        args = arguments("pbk_matmul")
        assert pbk.pbk_matmul(*args) == 0
        args[at] = one = Once()
        if error in (AttributeError, TypeError):
            assert binding._marshal.pbk_matmul(*args) is None and one.calls == 1
            continue
        with pytest.raises(error, match="once"):
            pbk.pbk_matmul(*args)
        assert one.calls == 1
