"""CPU-only checks of the C-ABI boundary: the library loads, exports every symbol
that include/iodf.h declares, and rejects malformed models on the host before any
GPU call is made."""
import ctypes
import os
import re

import numpy as np
import pytest

import paper_2206_08869_amd as iodf
from synth import CONFIGS, make_blob, parse_blob
from synth.model import pack_blob

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def _declared():
    text = open(os.path.join(ROOT, "include", "iodf.h")).read()
    text = re.sub(r"/\*.*?\*/", "", text, flags=re.S)
    return sorted(set(re.findall(r"\b(iodf_[a-z_]+)\s*\(", text)))


def test_library_exports_every_declared_symbol():
    lib = iodf.load_library()
    names = _declared()
    assert set(names) == set(iodf.EXPORTS)
    for n in names:
        assert getattr(lib, n) is not None


def test_strerror_covers_codes():
    lib = iodf.load_library()
    seen = {lib.iodf_strerror(c).decode() for c in range(0, -7, -1)}
    assert len(seen) == 7 and "unknown error" not in seen
    assert lib.iodf_strerror(-99).decode() == "unknown error"


def _init_code(blob, max_batch=1):
    lib = iodf.load_library()
    h = ctypes.c_void_p()
    blob = np.ascontiguousarray(blob, dtype=np.uint8)
    rc = lib.iodf_init(ctypes.byref(h), blob.ctypes.data_as(ctypes.c_void_p), blob.size, 0, max_batch)
    if rc == 0:
        lib.iodf_free(h)
    return rc


def test_init_rejects_bad_arguments_and_blobs_on_the_host():
    lib = iodf.load_library()
    good = make_blob(CONFIGS["cfg1"])
    assert lib.iodf_init(None, None, 0, 0, 1) == -1
    assert _init_code(good, max_batch=0) == -1
    bad = good.copy(); bad[4] ^= 0xFF
    assert _init_code(bad) == -2                                   # magic
    assert _init_code(good[:-8]) == -2                             # truncated
    assert _init_code(np.concatenate([good, np.zeros(4, np.uint8)])) == -2   # trailing bytes

    def edited(fn):
        m = parse_blob(good.copy())
        fn(m)
        return pack_blob(m)

    assert _init_code(edited(lambda m: m["nets"][0]["layers"][0]["shift"].__setitem__(0, 63))) == -2
    assert _init_code(edited(lambda m: m["nets"][0]["layers"][1]["M"].__setitem__(0, -1))) == -2
    assert _init_code(edited(lambda m: m["nets"][0]["layers"][0]["bias"].__setitem__(0, 1 << 30))) == -2
    assert _init_code(edited(lambda m: m["nets"][0]["perm"].__setitem__(0, int(m["nets"][0]["perm"][1])))) == -2
    assert _init_code(edited(lambda m: m["nets"][0]["layers"][0]["gate"].__setitem__(slice(None), 0))) == -2
    # well formed but not a valid flow: the translation channels may not be gated
    assert _init_code(edited(lambda m: m["nets"][0]["layers"][1]["gate"].__setitem__(0, 0))) == -3
    # unknown format flags in the header; an unsigned-format model whose hidden layer lacks a ReLU
    bad = good.copy(); bad[52] = 1
    assert _init_code(bad) == -2
    bad = good.copy(); bad[48] = 2
    assert _init_code(bad) == -2
    def unsigned_without_relu(m):
        m["act_unsigned"] = 1
        m["nets"][0]["layers"][0]["flags"] &= ~1
    assert _init_code(edited(unsigned_without_relu)) == -3
    # a filter whose 32-bit accumulator could overflow (Eq. 4-5): 3x3 over 16384 channels, all weights 127
    def overflowing(m):
        L0, L1 = m["nets"][0]["layers"]
        wide = 16384
        for key in ("bias", "M"):
            L0[key] = np.resize(L0[key], wide)
        L0["shift"] = np.resize(L0["shift"], wide); L0["gate"] = np.ones(wide, np.uint8)
        L0["W"] = np.zeros((wide,) + L0["W"].shape[1:], np.int8)
        L1["W"] = np.full((L1["W"].shape[0], wide, 3, 3), 127, np.int8)
    assert _init_code(edited(overflowing)) == -2
    def wide_but_small(m):
        overflowing(m)
        m["nets"][0]["layers"][1]["W"][:] = 1
    assert _init_code(edited(wide_but_small)) in (0, -5)             # accepted (no GPU here: the HIP error)
    # wrong number of networks for the declared structure
    assert _init_code(edited(lambda m: m["nets"].pop())) == -3
    # wrong wiring: second conv of a plain t() must read the first conv's width
    def narrow(m):
        L = m["nets"][0]["layers"][1]
        L["W"] = L["W"][:, :16]
    assert _init_code(edited(narrow)) == -3


def test_null_context_is_refused():
    lib = iodf.load_library()
    assert lib.iodf_forward(None, None, 1, None, None, None) == -1
    assert lib.iodf_inverse(None, None, 1, None, None) == -1
    v = ctypes.c_int64(0)
    assert lib.iodf_query(None, 0, ctypes.byref(v)) == -1
    lib.iodf_free(None)


def test_codec_tables_of_the_library_are_the_correctly_rounded_ones():
    # host-only entry point; the library builds its tables with its own code, the oracle with
    # its own, and the oracle's are pinned to 50-digit arithmetic elsewhere
    import oracle
    sig, inv = iodf.iodf_codec_tables()
    osig, oinv = oracle.prior_tables()
    assert np.array_equal(sig, osig) and np.array_equal(inv, oinv)
    lib = iodf.load_library()
    assert lib.iodf_codec_tables(None, None) == -1
    assert lib.iodf_encode(None, None, 1, None, 10, None, None) == -1
    assert lib.iodf_decode(None, None, 10, 1, None, None) == -1
    assert lib.iodf_prior_cf(None, None, None, 1, None, None, None) == -1
    # the single-layer probe checks its arguments before it touches the device
    assert lib.iodf_conv_probe(0, 0, 8, 3, 4, 4, 1, 1, None, None, None, None, None, None, 1, None) == -1
    assert lib.iodf_conv_probe(0, 8, 8, 2, 4, 4, 1, 1, None, None, None, None, None, None, 1, None) == -1
    # image sides beyond 8192 do not fit the kernels' argument block
    import ctypes
    buf = (ctypes.c_byte * 64)()
    assert lib.iodf_conv_probe(0, 8, 8, 3, 8193, 4, 1, 1, buf, buf, buf, buf, buf, buf, 1, None) == -1
    assert lib.iodf_conv_probe(0, 8, 8, 3, 4, 70000, 1, 1, buf, buf, buf, buf, buf, buf, 1, None) == -1
    assert lib.iodf_tile_patches(None, None, 8, 8, 0, 1, None, None) == -1


def test_recorded_traffic_is_tied_to_every_conv_source(tmp_path, monkeypatch):
    """bench.py reports recorded HBM traffic only for the build it was recorded with: any of the conv kernels' sources
    changes the hash."""
    import bench
    csrc = os.path.join(ROOT, "paper_2206_08869_amd", "csrc")
    assert {os.path.basename(f) for f in bench.CONV_SOURCES} == {f for f in os.listdir(csrc) if f.startswith("conv")}
    monkeypatch.setattr(bench, "ROOT", str(tmp_path))
    monkeypatch.setattr(bench, "CONV_SOURCES", ["a", "b", "c"])
    seen = set()
    for changed in ("", "a", "b", "c"):
        for f in "abc":
            (tmp_path / f).write_text("1" if f == changed else "0")
        seen.add(bench.conv_source_hash())
    assert len(seen) == 4
