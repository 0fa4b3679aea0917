"""The host encoder's 512-bit row loops against its 256-bit ones (which the oracle pins): the same bytes for every shape,
group, value kind and mask that either takes.  The 256-bit build is egt_host.cpp alone, without the 512-bit forms.  On a
processor without them the library takes the 256-bit loops too, and there is nothing to compare."""
import ctypes
import os
import shutil
import subprocess

import numpy as np
import pytest

from paper_2605_11582_amd import binding as B

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
# what egt_simd512::available() asks for, as /proc/cpuinfo names it
FEATURES = {"avx2", "f16c", "bmi2", "avx512f", "avx512bw", "avx512vl", "avx512dq", "avx512vbmi", "avx512_vbmi2"}
SYMBOLS = ("egt_status_str", "egt_2bitcsr_sizes", "egt_prune_n4", "egt_pack_2bitcsr", "egt_quant_int4")


@pytest.fixture(scope="module")
def narrow(tmp_path_factory):
    try:
        flags = next(line.split(":")[1].split() for line in open("/proc/cpuinfo") if line.startswith("flags"))
    except (OSError, StopIteration):
        flags = []
    if not FEATURES <= set(flags):
        pytest.skip("no 512-bit forms on this processor: " + ", ".join(sorted(FEATURES - set(flags))) + " missing")
    gxx = shutil.which("g++")
    if not gxx:
        pytest.skip("no host compiler")
    lib = str(tmp_path_factory.mktemp("host") / "libegt_host_256.so")
    build = subprocess.run([gxx, "-std=c++17", "-O1", "-fPIC", "-shared", "-pthread", "-ffp-contract=off", "-DEGT_HOST_AVX2_ONLY",
                            "-I" + os.path.join(ROOT, "include"), os.path.join(ROOT, "paper_2605_11582_amd", "csrc", "egt_host.cpp"), "-o", lib],
                           capture_output=True, text=True)
    assert build.returncode == 0, build.stderr
    return B._declare(ctypes.CDLL(lib), SYMBOLS)


def _weights(rng, rows, cols, form):
    if form == "bits":                                       # every binary16 number, infinities and NaN among them
        return rng.integers(0, 65536, (rows, cols)).astype(np.uint16).view(np.float16)
    if form == "ties":                                       # quotients that are half-integers, equal magnitudes, zeros of both signs
        w = (rng.integers(-9, 10, (rows, cols)) * 0.5 * 2.0 ** int(rng.integers(-24, 9))).astype(np.float16)
        w[rng.random(w.shape) < 0.2] = np.float16(-0.0)
        return w
    scale = {"subnormal": 2e-7, "ordinary": 0.02, "large": 2e4}[form]
    return np.clip(rng.standard_normal((rows, cols)) * scale, -65504, 65504).astype(np.float16)


def _all(w, seed):
    out = []
    rng = np.random.default_rng(seed)
    cols = w.shape[1]
    groups = [g for g in (4, 16, 32, 64, 96, 128, 192, cols) if cols % g == 0]
    for n in (1, 2, 3, 4):
        mask = B.prune_n4(w, n)
        out.append(mask)
        if seed % 2:
            mask = mask * (rng.random(mask.shape) < 0.7)         # groups that keep fewer
        mask = (mask.astype(np.uint8) * rng.integers(1, 256, mask.shape)).astype(np.uint8)     # any byte but zero keeps
        kept = np.where((mask != 0) & ~np.isfinite(w), np.float16(1.5), w)
        for kind in (B.VAL_INT4, B.VAL_INT4_PAIRED):
            for g in groups:
                p = B.pack_2bitcsr(kept, mask, n, g, kind)
                out += [p.row_ptr, p.values, p.idx, p.qparams]
        p = B.pack_2bitcsr(kept, mask, n, 0, B.VAL_FP16)
        out += [p.values, p.idx]
        bad = kept.copy()                                    # the first kept weight of the last row that keeps one
        bad[-1, int(np.argmax(mask[-1] != 0))] = np.float16(np.inf)
        with pytest.raises(B.EgtError) as e:
            B.pack_2bitcsr(bad, mask, n, 0, B.VAL_FP16)
        out.append(np.array([e.value.status]))
    if np.isfinite(w).all():
        for g in groups:
            out += list(B.quant_int4(w, g))
    return out


# (rows of 32 and 96 columns: not whole registers, all of them go to the 256-bit loops in either library)
@pytest.mark.parametrize("form", ["ordinary", "subnormal", "large", "ties", "bits"])
@pytest.mark.parametrize("cols", [32, 64, 96, 128, 192, 320, 1024])
def test_wide_and_narrow_row_loops_give_the_same_bytes(cols, form, narrow, monkeypatch):
    for seed in range(4):
        rng = np.random.default_rng(1000 * cols + seed)
        w = _weights(rng, int(rng.integers(1, 10)), cols, form)
        wide = _all(w, seed)
        with monkeypatch.context() as m:
            m.setattr(B, "_lib", narrow)
            slim = _all(w, seed)
        assert len(wide) == len(slim)
        for a, b in zip(wide, slim):
            assert np.asarray(a).tobytes() == np.asarray(b).tobytes()
