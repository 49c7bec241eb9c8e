"""The integer-only accumulation kernels (emulated FP64 and the fixed-point mode), the slicing and the GEMM kernels must contain
no FP64 instruction at all, and the hardware-FP64 accumulation kernel no FP64 multiply or fused multiply-add (the
product is formed on the matrix unit only).  Checked on the compiler's own assembly listing of the kernels (hipcc -S
cross-compiles without a GPU); a kernel's body runs from its label to its .Lfunc_end marker, so code behind an early
exit is inspected too."""
import os
import re
import subprocess

import pytest

import listing

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2508_00441_amd", "csrc")
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
F64 = r"\bv_\w*f64\w*"


_listings = {}


def _kernel_bodies(src, tmp_path):
    if src in _listings:
        return _listings[src]
    from paper_2508_00441_amd import build
    out = tmp_path / (src + ".s")
    flags = [f for f in build.FLAGS if f != "-fPIC"]
    subprocess.check_call([HIPCC] + flags + ["--cuda-device-only", "-S", os.path.join(CSRC, src), "-o", str(out)],
                          stdout=subprocess.DEVNULL, stderr=subprocess.DEVNULL)
    text = out.read_text()
    bodies = {}
    for m in re.finditer(r"^(_Z\w+):[^\n]*\n(.*?)^\.Lfunc_end\d+:", text, flags=re.S | re.M):
        bodies[m.group(1)] = m.group(2)
    _listings[src] = bodies
    return bodies


def _only(bodies, fragment):
    hit = [b for n, b in bodies.items() if fragment in n]
    assert len(hit) == 1, (fragment, [n for n in bodies if fragment in n])
    assert hit[0].count("s_endpgm") >= 1
    return hit[0]


@pytest.mark.skipif(not os.path.exists(HIPCC), reason="hipcc not available")
def test_integer_only_kernels_use_no_fp64(tmp_path):
    acc = _kernel_bodies("accumulate.hip", tmp_path)
    # accumulate_kernel<MODE, PINT>: MODE 0 hardware FP64, 1 emulated, 2 fixed point; PINT: INT32 products
    for pint in ("Lb0E", "Lb1E"):
        for mode in (1, 2):
            body = _only(acc, f"accumulate_kernelILi{mode}E{pint}")
            assert body.count("s_endpgm") >= 2                       # the early exit of a non-final pass and the normal one
            assert not re.search(F64, body), f"FP64 instruction in the integer-only accumulation kernel (mode {mode})"
        hw = _only(acc, f"accumulate_kernelILi0E{pint}")
        used = set(re.findall(r"\b(v_\w*f64\w*)", hw))
        assert used and all(re.match(r"v_(add|ldexp|cvt)_", u) for u in used), used      # adds, exponent scaling, converts only
    assert not re.search(F64, _only(acc, "axpby_kernelILb1E")), "FP64 instruction in the emulated scaling kernel"
    used = set(re.findall(r"\b(v_\w*f64\w*)", _only(acc, "axpby_kernelILb0E")))
    assert used and all(re.match(r"v_(add|mul)_f64", u) for u in used), used         # no fused multiply-add
    assert not re.search(F64, _only(acc, "add_emulated_kernel"))
    split = _kernel_bodies("split.hip", tmp_path)
    sk = [b for n, b in split.items() if "split_kernel" in n]
    assert len(sk) == 40              # 8 launch shapes x 5 slice formats
    stream = [b for n, b in split.items() if "split_stream_kernel" in n]
    assert len(stream) == 5
    for body in sk + stream:
        assert not re.search(F64, body), "FP64 instruction in a slicing kernel"
    gemm = _kernel_bodies("pair_gemm.hip", tmp_path)
    assert len(gemm) == 5
    for n, body in gemm.items():
        assert not re.search(F64, body)
        assert "v_mfma_f32_32x32x64_f8f6f4" in body or "v_mfma_f32_32x32x16_f16" in body or "v_mfma_i32_32x32x32_i8" in body


@pytest.mark.skipif(not os.path.exists(HIPCC), reason="hipcc not available")
def test_the_other_integer_only_kernels_use_no_fp64(tmp_path):
    """The forms for few elements and for scaled calls, short and long blocks, and the other GEMM kernels."""
    acc = _kernel_bodies("accumulate.hip", tmp_path)
    for name in ("accumulate_fine_kernel", "accumulate_scaled_kernel", "accumulate_scaled_fine_kernel"):
        for pint in ("Lb0E", "Lb1E"):
            for mode in (1, 2):
                assert not re.search(F64, _only(acc, f"{name}ILi{mode}E{pint}")), (name, mode, pint)
            used = set(re.findall(r"\b(v_\w*f64\w*)", _only(acc, f"{name}ILi0E{pint}")))
            ops = "add|ldexp|cvt|mul" if "scaled" in name else "add|ldexp|cvt"
            assert used and all(re.match(rf"v_({ops})_", u) for u in used), used         # no fused multiply-add
    split = _kernel_bodies("split.hip", tmp_path)
    short = [b for n, b in split.items() if "slice_short_kernel" in n]
    assert len(short) == 4
    for body in short + [_only(split, "long_exponents_kernel"), _only(split, "delta_kernel")]:
        assert not re.search(F64, body), "FP64 instruction in a slicing kernel"
    for source, kernels, mfma in (("pair_gemm_fp8.hip", 2, r"v_mfma_f32_16x16x128_f8f6f4"), ("pair_gemm_measured.hip", None, r"v_mfma_"), ("pair_gemm_small.hip", None, r"v_mfma_")):
        gemm = {n: b for n, b in _kernel_bodies(source, tmp_path).items() if "pair_gemm" in n}
        assert gemm and (kernels is None or len(gemm) == kernels)
        for n, body in gemm.items():
            assert not re.search(F64, body), n
            assert re.search(mfma, body), n


@pytest.mark.skipif(not listing.AVAILABLE, reason="no LLVM tools")
def test_no_integer_only_kernel_of_the_library_uses_fp64():
    """Every kernel of the built library: the one pass over all pairs and the vectors off its ladder in all formats, slice counts and parts, the forms
    behind it, and all the others."""
    seen = {}
    for symbol, text in listing.texts().items():
        used = set(re.findall(r"^\s+(v_\w*f64\w*)", text, flags=re.M))
        name = re.search(r"\d+([a-z_0-9]+_kernel)", symbol).group(1)
        # the kernels with a mode: its place among the template arguments, and the value of the hardware sum
        at, hardware = {"ladder_sums_kernel": (2, "0"), "off_ladder_kernel": (2, "0"), "axpby_kernel": (0, "0")}.get(name, (0, "0") if name.startswith("accumulate_") else (None, None))
        if at is not None and re.findall(r"L[ib](\d+)E", symbol)[at] == hardware:
            seen[name, "hw"] = seen.get((name, "hw"), 0) + 1
            assert used and all(re.match(r"v_(add|ldexp|cvt|mul)_", u) for u in used), (symbol, used)      # no fused multiply-add
        else:
            seen[name, ""] = seen.get((name, ""), 0) + 1
            assert not used, (symbol, used)
    for name in ("accumulate_kernel", "accumulate_fine_kernel", "accumulate_rest_kernel", "accumulate_fine_rest_kernel", "accumulate_scaled_kernel",
                 "accumulate_scaled_fine_kernel", "accumulate_scaled_rest_kernel", "accumulate_scaled_fine_rest_kernel"):
        assert seen[name, "hw"] == 2 and seen[name, ""] == 4, name    # INT32 and FP32 products
    assert seen["off_ladder_kernel", "hw"] == seen["off_ladder_kernel", ""] == 14        # FP8 with 6 to 13 slices, INT8 with 6 to 11
    assert seen["ladder_sums_kernel", ""] > seen["ladder_sums_kernel", "hw"] >= 40
    assert seen["pair_gemm_small_kernel", ""] == 10 and seen["split_kernel", ""] == 40 and seen["slice_short_kernel", ""] == 4
