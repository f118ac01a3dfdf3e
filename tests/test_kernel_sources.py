"""Properties of the device code that no run on a GPU shows: read from the sources and from the code generated for them."""
import os
import re

import pytest

from paper_2605_28657_amd import build as b

KERNELS = [s for s in b.SOURCES if s.startswith("kernels_")]


def _calls(text, name):
    """(position, arguments) of every call of `name` in the text."""
    for m in re.finditer(re.escape(name.rstrip("(")) + r"\w*\(", text):
        depth, args, cur = 1, [], ""
        for ch in text[m.end():]:
            depth += (ch in "([{") - (ch in ")]}")
            if depth == 0:
                break
            if ch == "," and depth == 1:
                args.append(cur.strip())
                cur = ""
            else:
                cur += ch
        yield m.start(), args + [cur.strip()]


@pytest.mark.parametrize("src", KERNELS)
def test_scalar_offsets_stay_inside_the_descriptor(src):
    """A buffer load's range check covers the per-lane offset only: it is compared with (size - scalar offset), which means
    nothing once the scalar offset is past the size.  Prefetches run past a layer's last weight block, so every load
    with a scalar offset must go through a descriptor that reaches over the slack (weight_rsrc)."""
    text = open(os.path.join(b.CSRC, src)).read()
    kernels = [m.start() for m in re.finditer(r"__global__", text)] + [len(text)]
    loads = 0
    for pos, args in _calls(text, "__builtin_amdgcn_raw_buffer_load"):
        assert len(args) == 4, (src, args)
        if args[2] == "0":
            continue
        kernel = text[max(k for k in kernels if k < pos):min(k for k in kernels if k > pos)]
        # the descriptor itself, or a parameter of the lambda that every caller fills with one
        if args[0] == "rs":
            made = [a[1] for _, a in _calls(kernel, "load_set(") if a[1].startswith("rs_")]
            assert made
        else:
            made = [args[0]]
        for rs in made:
            assert re.search(rf"\b{rs} = weight_rsrc\(", kernel), f"{src}: {rs} takes a scalar offset {args[2]!r} but covers no slack"
        loads += 1
    if loads:
        assert "kWeightSlack" in text or "if (more) load_a(stage + 1);" in text, f"{src}: how far its prefetch runs is not checked"


def test_the_parameter_allocation_ends_with_the_slack():
    text = open(os.path.join(b.CSRC, "api.hip")).read()
    assert re.search(r"ar\.reserve\(kWeightSlack\);\s*hipError_t e = hipMalloc\(&v->d_params, ar\.bytes\.size\(\)\)", text)


def test_surplus_pieces_of_sums_in_parts_stay_out_of_range():
    """The offset of a tile's surplus piece, scaled to rows of sums, lies past every descriptor the launch accepts; other offsets are the
    row's, as far as a window's sums reach."""
    import ctypes
    import subprocess
    import tempfile
    text = open(os.path.join(b.CSRC, "conv_bf16.h")).read()
    stream = open(os.path.join(b.CSRC, "kernels_bf16_stream.hip")).read()
    (parts,) = re.findall(r"constexpr int kConvParts = (\d+);", open(os.path.join(b.CSRC, "internal.h")).read())
    (limit,) = re.findall(r"max_out_bytes > (0x\w+)ll\) return hipErrorInvalidValue;", open(os.path.join(b.CSRC, "kernels_bf16.hip")).read())
    parts, limit = int(parts), int(limit, 16)
    assert "part_voff(off, (unsigned)ec)" in stream and "return kOutOfRange;" in stream
    out_of_range = int(re.search(r"kOutOfRange = (0x\w+)u;", text).group(1), 16)
    fn = re.search(r"__host__ __device__ (constexpr unsigned part_voff\(.*?\n})", text, re.S).group(1)
    with tempfile.TemporaryDirectory() as d:
        src, lib = os.path.join(d, "f.cpp"), os.path.join(d, "f.so")
        open(src, "w").write(f"constexpr int kConvParts = {parts};\nconstexpr unsigned kOutOfRange = {out_of_range}u;\n{fn}\n"
                             "extern \"C\" unsigned f(unsigned off, unsigned ch) { return part_voff(off, ch); }\n")
        subprocess.run(["g++", "-std=c++17", "-shared", "-fPIC", "-o", lib, src], check=True)
        f = ctypes.CDLL(lib).f
        f.restype, f.argtypes = ctypes.c_uint, [ctypes.c_uint, ctypes.c_uint]
        for cout in (128, 256):
            last = limit // (4 * parts * cout) - 1                      # last row of the largest window
            for ch in range(0, cout, 8):
                assert f(out_of_range, ch) >= limit
                for row in (0, 1, 97, last - 1, last, last + 127):      # a tile's columns run past the last row
                    at = f((row * cout + ch) * 2, ch)
                    assert at == row * parts * cout * 4 + ch * 4 and (row <= last) == (at + 32 <= limit)


def _resources(fields=("private_segment_fixed_size", "vgpr_spill_count")):
    """{kernel: (bytes of scratch memory, spilled registers)}, or other fields, of the gfx950 code in the built library."""
    import subprocess
    import tempfile
    llvm = "/opt/rocm/llvm/bin"
    if not (os.path.exists(b.LIB) and os.path.exists(os.path.join(llvm, "llvm-readelf"))):
        pytest.skip("no built library or no LLVM tools")
    out = {}
    with tempfile.TemporaryDirectory() as d:
        fat, one, elf = (os.path.join(d, n) for n in ("fat", "one", "elf"))
        subprocess.run([f"{llvm}/llvm-objcopy", f"--dump-section=.hip_fatbin={fat}", b.LIB, os.path.join(d, "copy")], check=True)
        data = open(fat, "rb").read()
        starts = [m.start() for m in re.finditer(b"__CLANG_OFFLOAD_BUNDLE__", data)] + [len(data)]
        for lo, hi in zip(starts, starts[1:]):
            open(one, "wb").write(data[lo:hi])
            subprocess.run([f"{llvm}/clang-offload-bundler", "--unbundle", "--type=o", f"--input={one}", f"--output={elf}",
                            "--targets=hipv4-amdgcn-amd-amdhsa--gfx950"], check=True)
            notes = subprocess.run([f"{llvm}/llvm-readelf", "--notes", elf], capture_output=True, text=True, check=True).stdout
            for k in notes.split("- .agpr_count:")[1:]:
                field = lambda f: re.search(rf"\.{f}:\s+(\S+)", k).group(1)
                out[field("name")] = tuple(int(field(f)) for f in fields)
    return out


def test_convolution_kernels_keep_their_accumulators_in_registers():
    """A dynamic index into the accumulators puts them in scratch memory, a round trip per stage of the K loop."""
    res = {n: r for n, r in _resources().items() if "conv_" in n or "res_unit_wide" in n or "res_unit_narrow" in n}
    assert len(res) > 100
    assert {n: r for n, r in res.items() if r != (0, 0)} == {}


def test_kernel_arguments_do_not_grow():
    """The host bounds a call of empty launches (a gated call whose clips are skipped), and issues the launches with longer arguments later."""
    limit = {"conv_stream_kernel": 144, "conv_tall_kernel": 144, "conv_mfma_kernel": 128, "res_unit_fused_kernel": 456,
             "res_unit_narrow_stream_kernel": 456, "res_unit_wide": 376}
    seen = set()
    for name, (size,) in _resources(("kernarg_segment_size",)).items():
        for k, most in limit.items():
            if re.search(rf"\d{k}", name):
                seen.add(k)
                assert size <= most, (name, size)
    assert seen == set(limit)


def test_descriptors_are_scalar():
    """A buffer descriptor held in vector registers turns every load through it into a loop over the lanes' values
    (v_readfirstlane of all four words, a compare, a branch back)."""
    import shutil
    import subprocess
    import tempfile
    from concurrent.futures import ThreadPoolExecutor
    if shutil.which("hipcc") is None:
        pytest.skip("hipcc not available")
    flags = [f for f in b.FLAGS if f != "-fPIC"]

    def asm_of(src):
        with tempfile.TemporaryDirectory() as d:
            out = os.path.join(d, "k.s")
            subprocess.run(["hipcc"] + flags + ["-S", "--cuda-device-only", "-o", out, os.path.join(b.CSRC, src)], check=True, capture_output=True)
            return open(out).read()

    srcs = ["kernels_bf16_stream.hip", "kernels_bf16.hip", "kernels_bf16_wide.hip", "kernels_bf16_fused.hip", "kernels_f32.hip"]
    with ThreadPoolExecutor(max_workers=len(srcs)) as ex:
        for src, text in zip(srcs, ex.map(asm_of, srcs)):
            # the loop's mark: descriptor words compared with the lanes' own, then the lanes that agree masked in
            loops = re.findall(r"v_cmp_eq_u64_e\w+ [^\n]*\n(?:[^\n]*\n){0,8}?[^\n]*s_and_saveexec_b64", text)
            assert not loops, f"{src}: {len(loops)} loops over a descriptor's lanes"
