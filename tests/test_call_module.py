"""_pwlq_call hands every argument of the one-tensor calls to the library's function as ctypes does (no GPU): the function
called is a recorder with that function's signature."""
import ctypes

import numpy as np
import pytest

torch = pytest.importorskip("torch")
from paper_2002_00104_amd import _pwlq_call, pwlq  # noqa: E402

VP, I64, CI, SZ, CF = ctypes.c_void_p, ctypes.c_int64, ctypes.c_int, ctypes.c_size_t, ctypes.c_float
SIGNATURES = {
    "search": [VP, I64, I64, CI, CI, CI, VP, VP, VP, VP, VP, SZ, VP],
    "quantize": [VP, I64, I64, CI, CI, VP, VP, VP, VP, VP, VP],
    "linear_i8": [VP, I64, I64, CF, CF, VP, VP, I64, CI, VP, VP, VP, VP, VP, SZ, VP],
}


def recorder(types, got, status):
    def f(*args):
        got[:] = args
        return status
    return ctypes.CFUNCTYPE(CI, *types)(f)


def test_the_signatures_are_the_library_s():
    for name, functions in (("search", ("pwlq_search", "pwlq_search_fast")), ("quantize", ("pwlq_quantize", "pwlq_quantize_packed")),
                            ("linear_i8", ("pwlq_linear_i8",))):
        for f in functions:
            assert getattr(pwlq.lib, f).argtypes == SIGNATURES[name], f


# pointers that the library takes as NULL or that are handles: everything else has to be a tensor
OPTIONAL = {"search": [], "quantize": [9], "linear_i8": [12]}
STREAM = {"search": 12, "quantize": 10, "linear_i8": 15}


@pytest.mark.parametrize("name", list(SIGNATURES))
@pytest.mark.parametrize("seed", [1, 2, 3])
def test_every_argument_arrives_in_its_place(name, seed):
    types, got, rng = SIGNATURES[name], [], np.random.default_rng(seed)
    keep, args, want = [], [], []
    for i, t in enumerate(types):
        if t is VP:
            if i in OPTIONAL[name] and seed % 2:
                args.append(None)
                want.append(None)
            elif i == STREAM[name]:
                args.append(int(rng.integers(1, 1 << 47)) if seed < 3 else 0)
                want.append(args[-1] or None)
            else:
                keep.append(torch.empty(int(rng.integers(1, 50))))
                args.append(keep[-1])
                want.append(keep[-1].data_ptr())
        elif t is CF:
            args.append(int(rng.integers(-9, 9)) if (i + seed) % 2 else float(rng.standard_normal()))
            want.append(float(np.float32(args[-1])))
        else:
            bound = 1 << (30 if t is CI else 62)
            args.append(np.int64(rng.integers(0 if t is SZ else -bound, bound)) if seed == 2 else int(rng.integers(0 if t is SZ else -bound, bound)))
            want.append(int(args[-1]))
    fn = recorder(types, got, 7 * seed)
    assert getattr(_pwlq_call, name)(ctypes.cast(fn, VP).value, *args) == 7 * seed
    assert got == want


@pytest.mark.parametrize("name", list(SIGNATURES))
def test_an_address_is_taken_for_the_stream_alone(name):
    """An integer in the place of a tensor (a width for a parameter) would reach a kernel as a device address."""
    types, got = SIGNATURES[name], []
    fn = ctypes.cast(recorder(types, got, 0), VP).value
    t = torch.empty(4)
    good = [t if x is VP else 1 for x in types]
    good[STREAM[name]] = 0
    for i, x in enumerate(types):
        if x is not VP or i == STREAM[name]:
            continue
        for value in [16, 0, True, 1 << 40, np.int64(16)] + [None] * (i not in OPTIONAL[name]):
            with pytest.raises(AttributeError):
                getattr(_pwlq_call, name)(fn, *good[:i], value, *good[i + 1:])
    for value in (None, t, 1.5):
        with pytest.raises(TypeError):
            getattr(_pwlq_call, name)(fn, *good[:-1], value)
        with pytest.raises(TypeError):
            getattr(_pwlq_call, name)(value, *good)
    with pytest.raises(TypeError):
        getattr(_pwlq_call, name)(0, *good)
    assert got == []
    assert getattr(_pwlq_call, name)(fn, *good) == 0 and got[0] == t.data_ptr()


def test_what_is_no_argument_is_refused_before_the_call():
    got = []
    fn = recorder(SIGNATURES["quantize"], got, 0)
    t = torch.empty(4)
    good = [ctypes.cast(fn, VP).value, t, 1, 1, 4, 0, t, t, t, t, None, 0]
    for at, value, error in ((1, 1.5, AttributeError), (2, 1.5, TypeError), (2, 1 << 70, OverflowError), (4, 1 << 40, OverflowError),
                             (4, None, TypeError), (8, "x", AttributeError), (11, 1 << 70, OverflowError)):
        with pytest.raises(error):
            _pwlq_call.quantize(*good[:at], value, *good[at + 1:])
    with pytest.raises(TypeError):
        _pwlq_call.quantize(*good[:-1])
    assert got == []
    assert _pwlq_call.quantize(*good) == 0 and got[0] == t.data_ptr()
