"""csrc/bind.cpp: what it leaves to the way through ctypes (on the host), and that what it takes reaches the C ABI as that way would
hand it over (on the GPU: entry points that note their arguments stand in for the library's)."""
import ctypes

import numpy as np
import pytest
import torch

from paper_2504_18154_amd import binding

fast = binding._fast
BF, I32 = torch.bfloat16, torch.int32


def _args(device):
    rows = torch.zeros(3, 12, 16, dtype=BF, device=device)  # [tokens, 8 + 2 + 2 heads, 16]
    a = {"q": rows[:, :8], "kn": rows[:, 8:10], "vn": rows[:, 10:], "kc": torch.zeros(99, dtype=BF, device=device), "vc": torch.zeros(99, dtype=BF, device=device),
         "bt": torch.zeros(2, 7, dtype=I32, device=device), "len": torch.zeros(2, dtype=I32, device=device), "cu": torch.zeros(3, dtype=I32, device=device),
         "out": torch.zeros(3, 8, 16, dtype=BF, device=device), "lse": torch.zeros(3, 8, device=device)}
    return a


def _calls(a, most, handle=77):
    return {"kv_append": (handle, a["kc"], a["vc"], a["kn"], a["vn"], a["cu"], a["len"], a["bt"], most, 0),
            "attn_prefill": (handle, a["q"], a["kc"], a["vc"], a["cu"], a["len"], a["bt"], a["out"], a["lse"], most, 0),
            "attn_decode": (handle, a["q"], a["kc"], a["vc"], a["bt"], a["len"], a["out"], most, a["lse"], 0),
            "attn_decode_append": (handle, a["q"], a["kn"], a["vn"], a["kc"], a["vc"], a["bt"], a["len"], a["out"], most, a["lse"]),
            "attn_decode_noalloc": (0, handle, a["q"], a["kc"], a["vc"], a["bt"], a["len"], a["out"], most, a["lse"])}


@pytest.mark.parametrize("change", [{"q": np.zeros((3, 8, 16))}, {"kc": "pool"}, {"len": [1, 2]}, {"bt": torch.zeros(7, dtype=I32)}, {"bt": None},
                                    {"len": None}, {"most": 3.0}, {"most": np.int32(3)}, {"most": True}, {"most": 1 << 31}, {"most": 1 << 70}, {"handle": None},
                                    {"q": torch.zeros(3, 8, dtype=BF)}, {"q": torch.zeros(3, 16, 8, dtype=BF).transpose(1, 2)}, {"vn": torch.zeros(3, 2, 16, dtype=BF)}],
                         ids=str)
def test_what_is_left_to_the_other_way(change):
    a = _args("cpu")
    plain = {k: _calls(a, 3)[k] for k in _calls(a, 3)}
    a.update({k: v for k, v in change.items() if k in a})
    changed = _calls(a, change.get("most", 3), change.get("handle", 77))
    touched = [k for k in plain if any(x is not y for x, y in zip(plain[k], changed[k]))]
    strides = {"q": ("attn_prefill", "attn_decode", "attn_decode_append"), "vn": ("kv_append", "attn_decode_append")}
    if "q" in change and torch.is_tensor(change["q"]):
        touched = strides["q"]
    if "vn" in change:
        touched = strides["vn"]
    assert touched
    for name in touched:
        assert getattr(fast, name)(*changed[name]) == -1, name
    assert fast.kv_append(1, 2) == -1  # (too few)


@pytest.mark.gpu
def test_what_reaches_the_c_abi():
    vp, i32, i64 = ctypes.c_void_p, ctypes.c_int32, ctypes.c_int64
    a = _args("cuda")
    p = {k: v.data_ptr() for k, v in a.items()}
    s = torch.cuda.current_stream().cuda_stream or None
    side = torch.cuda.Stream()
    types = {"kv_append": [vp, vp, vp, vp, vp, i64, vp, vp, vp, i32, i32, i32, i32, vp],
             "attn_prefill": [vp, vp, i64, vp, vp, vp, vp, vp, i32, vp, vp, i32, i32, i32, vp],
             "attn_decode": [vp, vp, i64, vp, vp, vp, i32, vp, vp, vp, i32, i32, vp],
             "attn_decode_append": [vp, vp, i64, vp, vp, i64, vp, vp, vp, i32, vp, vp, vp, i32, i32, vp],
             "attn_decode_noalloc": [ctypes.c_int, vp, vp, vp, vp, vp, i32, vp, vp, vp, i32, i32, vp]}
    seen = {}

    def note(name):
        def f(*args):
            seen[name] = args
            return 3
        return ctypes.CFUNCTYPE(ctypes.c_int, *types[name])(f)

    stand_ins = {k: note(k) for k in types}

    def expected(stream, lse, packed):
        kv, q = (32, 128) if packed else (192, 192)
        return {"kv_append": (77, p["kc"], p["vc"], p["kn"], p["vn"], kv, p["cu"], p["len"], p["bt"], 7, 2, 3, 3, stream),
                "attn_prefill": (77, p["q"], q, p["kc"], p["vc"], p["cu"], p["len"], p["bt"], 7, p["out"], lse, 2, 3, 3, stream),
                "attn_decode": (77, p["q"], q, p["kc"], p["vc"], p["bt"], 7, p["len"], p["out"], lse, 2, 40, stream),
                "attn_decode_append": (77, p["q"], 192, p["kn"], p["vn"], 192, p["kc"], p["vc"], p["bt"], 7, p["len"], p["out"], lse, 2, 40, stream),
                "attn_decode_noalloc": (0, 77, p["q"], p["kc"], p["vc"], p["bt"], 7, p["len"], p["out"], lse, 2, 40, stream)}

    try:
        fast.bind(*(ctypes.cast(stand_ins[k], vp).value for k in types))
        for stream, handle in ((None, s), (side, side.cuda_stream)):
            for lse in (a["lse"], None):
                for packed in (False, True):
                    b = dict(a, lse=lse)
                    calls = _calls(b, 40)
                    calls["kv_append"] = calls["kv_append"][:8] + (None, 32 if packed else 0)  # (None: all the tokens)
                    calls["attn_prefill"] = calls["attn_prefill"][:9] + (None, 128 if packed else 0)
                    calls["attn_decode"] = calls["attn_decode"][:9] + (128 if packed else 0,)
                    want = expected(handle, p["lse"] if lse is not None else None, packed)
                    with torch.cuda.stream(stream):
                        for name in types:
                            assert getattr(fast, name)(*calls[name]) == 3
                            assert seen.pop(name) == want[name], name
    finally:
        lib = binding._lib
        fast.bind(*(ctypes.cast(f, vp).value for f in (lib.ecoserve_kv_append_strided, lib.ecoserve_attn_prefill_strided, lib.ecoserve_attn_decode_strided,
                                                       lib.ecoserve_attn_decode_append, lib.ecoserve_attn_decode_noalloc)))


def test_a_library_for_another_torch_is_not_current(monkeypatch):
    """Built for another torch _bind.so does not load, and what the error says to run must then build it."""
    from paper_2504_18154_amd import build
    monkeypatch.setattr(build, "_deps_mtime", lambda: 0.0)
    assert build.is_current() and build._bind_fits() in fast.__doc__
    monkeypatch.setattr(torch, "__version__", "0.0.0")
    assert not build.is_current()


@pytest.mark.parametrize("bound", [np.int32(40), np.int64(40), torch.tensor(40), 40.0, 40], ids=["int32", "int64", "tensor", "float", "int"])
def test_bounds_that_are_no_plain_integers_take_the_usual_way(bound, monkeypatch):
    """lens.max() of an array is a bound like any other: the hot calls hand it over as an integer."""
    class Noted:
        def __getattr__(self, name):
            return lambda *args: seen.update({name: args}) or (0 if type(args[at[name]]) in (int, type(None)) else -1)

    monkeypatch.setattr(binding, "_fast", Noted())
    c = object.__new__(binding.Context)
    c._address, c._h, c._q_row, c._kv_row = 77, None, 128, 32
    at = {"kv_append": 8, "attn_prefill": 9, "attn_decode": 7, "attn_decode_append": 9, "attn_decode_noalloc": 8}
    t = [None] * 7
    for call, name in ((lambda: c.kv_append(*t, bound), "kv_append"), (lambda: c.kv_append_strided(*t, bound), "kv_append"),
                       (lambda: c.attn_prefill(*t, None, bound), "attn_prefill"), (lambda: c.attn_prefill_strided(*t, None, bound), "attn_prefill"),
                       (lambda: c.attn_decode(*t[:6], bound), "attn_decode"), (lambda: c.attn_decode_strided(*t[:6], bound), "attn_decode"),
                       (lambda: c.attn_decode_append(*t, None, bound), "attn_decode_append"),
                       (lambda: binding.attn_decode_noalloc(binding.Layout(), *t[:6], bound), "attn_decode_noalloc")):
        seen = {}
        call()
        assert type(seen[name][at[name]]) is int and seen[name][at[name]] == 40, name
    seen = {}
    c.kv_append(*t)
    c.attn_prefill(*t)
    assert seen["kv_append"][8] is None and seen["attn_prefill"][9] is None   # (all the tokens)
