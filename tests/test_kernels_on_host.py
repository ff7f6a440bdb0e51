"""The depthwise-convolution and attention kernels and the contractions straight from the caller's tensors
(gemm_any.hip, gemm_any_f64.hip, gemm_exact.hip) run on the host, thread by thread, under the address
and undefined-behaviour sanitizers: every global and LDS access of launch geometries like the GPU tests'
is checked against exactly sized buffers, and the results against float64 loops in the drivers.  The
kernels' source is taken as it is (HIP headers replaced by a small vocabulary header, launchers cut off,
instructions of a whole wavefront replaced by their stand-ins)."""
import os
import re
import subprocess

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(ROOT, "paper_2203_15952_amd", "csrc")


def spliced_source():
    src = open(os.path.join(CSRC, "conv.hip")).read()
    epi = open(os.path.join(CSRC, "epilogue.h")).read()
    epi = epi.replace("#include <hip/hip_runtime.h>", "").replace("#pragma once", "")
    assert '#include "aqt_internal.h"' in src and '#include "epilogue.h"' in src
    src = src.replace('#include "aqt_internal.h"', '#include "hip_on_host.h"').replace('#include "epilogue.h"', epi)
    assert src.count("extern __shared__ float lds[];") == 2
    src = src.replace("extern __shared__ float lds[];", "AQT_EXTERN_LDS(lds);")
    src = src[:src.index("aqt_status launch_corr")]          # kernels and geometry helpers only
    return src + open(os.path.join(HERE, "host_emulation", "conv_driver.cpp")).read()


def spliced_attention_source(driver="attention_driver.cpp"):
    src = open(os.path.join(CSRC, "attention.hip")).read()
    src = src.replace('#include "aqt_internal.h"', '#include "hip_on_host.h"')
    vec = "typedef float v4f __attribute__((ext_vector_type(4)));"      # a clang extension; g++ gets a plain struct
    assert vec in src
    src = src.replace(vec, "struct alignas(16) v4f { float x, y, z, w; };")
    vec16 = "typedef float v16f __attribute__((ext_vector_type(16)));"                # the shim has its own
    assert vec16 in src
    src = src.replace(vec16, "")
    src = src[:src.index("}  // namespace\n\nbool attention_shape_ok")]  # kernel and geometry helper only
    return src + open(os.path.join(HERE, "host_emulation", driver)).read()


def cut(src, start, end):
    """src without what lies between two of its lines (start included, end not)."""
    i = src.index(start)
    return src[:i] + src[src.index(end, i):]


def read(name):
    src = open(os.path.join(CSRC, name)).read()
    src = re.sub(r"^ *typedef \w+ v\w+ __attribute__\(\(ext_vector_type\(\d+\)\)\);\n", "", src, flags=re.M)   # structs in the shim
    return re.sub(r"^#(include|pragma once).*\n", "", src, flags=re.M)


def bf16_terms():
    """bf16_terms.h without what the shim stands in for: the conversion and the matrix instruction."""
    src = cut(read("bf16_terms.h"), "__device__ __forceinline__ uint32_t pack_bf16", "__device__ __forceinline__ v16f mfma_bf16")
    return cut(src, "__device__ __forceinline__ v16f mfma_bf16", "// hi = bf16(a), lo")


def spliced_attention_rows_source():
    shape = open(os.path.join(CSRC, "aqt_internal.h")).read()
    shape = shape[shape.index("struct AttnShape {"):]
    shape = shape[:shape.index("};") + 2]
    tiles = read("attention_tiles.h").replace("namespace aqt {", "namespace aqt {\n" + shape, 1)
    fwd = read("attention_fwd.hip").replace("namespace aqt {\nnamespace {", "namespace aqt {\nnamespace fwd_rows {")
    fwd = fwd[:fwd.index("aqt_status launch_attention_rows")] + "}\n"
    few = read("attention_few.hip").replace("namespace aqt {\nnamespace {", "namespace aqt {\nnamespace few {")
    few = few[:few.index("}  // namespace\n\n// As long as all of its workgroups")] + "}\n}\n"
    bwd = read("attention_bwd.hip").replace("namespace aqt {\nnamespace {", "namespace aqt {\nnamespace bwd_rows {")
    bwd = bwd[:bwd.index("bool attention_rows_ok")] + "}\n"
    # instructions that the shim stands in for
    bwd = cut(bwd, "  typedef __attribute__((address_space(3)))", "  return v4i{a.x, a.y, b.x, b.y};")
    bwd = bwd.replace("  return v4i{a.x, a.y, b.x, b.y};", "  const v2i a = read_tr_b16(at + AT), b = read_tr_b16(at + AT + 8 * kRowBytes);\n  return v4i{a.x, a.y, b.x, b.y};")
    bwd = bwd.replace("v4i read_tr8(uint32_t at)", "v4i read_tr8(const uint8_t *at)")
    bwd = bwd.replace("const uint32_t at = static_cast<uint32_t>(reinterpret_cast<uintptr_t>(tensor))", "const uint8_t *const at = tensor")
    assert bwd.count('asm volatile("" : "+') == 2
    bwd = re.sub(r' *asm volatile\("" : "\+[sv]"\(\w+\)\);\n', "", bwd)
    driver = open(os.path.join(HERE, "host_emulation", "attention_rows_driver.cpp")).read()
    return '#include "vectors_on_host.h"\n' + bf16_terms() + tiles + fwd + few + bwd + driver


def spliced_gemm_any_source():
    any_ = read("gemm_any.hip").replace("namespace aqt {\nnamespace {", "namespace aqt {\nnamespace any {")
    fill = any_[any_.index("// ---- forward from float32 rows"):any_.index("template <int TM, int TN, int WM, int WN, int WK, int BK, bool PACKED>\naqt_status")]
    any_ = any_[:any_.index("// Which workgroup arrangement of the forward.")] + fill + "}\n}\n"
    internal = open(os.path.join(CSRC, "aqt_internal.h")).read()
    sources = "".join(internal[i:internal.index("};", i) + 2] + "\n" for i in (internal.index("struct RowSource {"), internal.index("struct DenseSource {\n")))
    slabs = re.search(r"^constexpr int kWeightSlabs = .*$", internal, flags=re.M).group(0)
    quant = read("quant_code.h") + "namespace aqt {\n" + slabs + "\n" + sources + "}\n"
    f64 = read("gemm_any_f64.hip").replace("namespace aqt {\nnamespace {", "namespace aqt {\nnamespace f64 {")
    f64 = f64[:f64.index("template <int TN, int WN, int WK, bool PACKED, int MODE>\naqt_status")] + "}\n}\n"
    exact = read("gemm_exact.hip").replace("namespace aqt {\nnamespace {", "namespace aqt {\nnamespace exact {")
    exact = exact[:exact.index("// Tiles of at most five blocks of sixteen")] + "}\n}\n"
    exact = cut(exact, "__device__ __forceinline__ float load_f32", "__device__ __forceinline__ double power_of_two")   # the shim has its own
    driver = open(os.path.join(HERE, "host_emulation", "gemm_any_driver.cpp")).read()
    return ('#include "vectors_on_host.h"\n#include "aqt.h"\n' + read("any_shape.h") + bf16_terms() + read("colsum.h") +
            read("epilogue.h") + quant + any_ + f64 + exact + driver)


def test_lanes_hand_over_lds_behind_fences():
    """A scheduling barrier alone states no order of memory: every hand-over inside a wavefront goes through wave_lds_order."""
    sources = {f: open(os.path.join(CSRC, f)).read() for f in sorted(os.listdir(CSRC)) if f.endswith((".hip", ".h"))}
    assert [f for f, src in sources.items() if "__builtin_amdgcn_wave_barrier" in src] == ["aqt_internal.h"]
    assert re.search(r'fence\(__ATOMIC_RELEASE, "wavefront"\);\s+__builtin_amdgcn_wave_barrier\(\);\s+__builtin_amdgcn_fence\('
                     r'__ATOMIC_ACQUIRE, "wavefront"\);', sources["aqt_internal.h"])


def test_conv_kernels_in_bounds_and_correct_on_host(tmp_path):
    build_and_run(tmp_path, "conv_on_host", spliced_source())


def test_attention_kernel_in_bounds_and_correct_on_host(tmp_path):
    build_and_run(tmp_path, "attention_on_host", spliced_attention_source())


def test_attention_backward_kernels_in_bounds_and_correct_on_host(tmp_path):
    build_and_run(tmp_path, "attention_bwd_on_host", spliced_attention_source("attention_bwd_driver.cpp"))


def test_attention_kernels_for_vectorised_rows_in_bounds_and_correct_on_host(tmp_path):
    build_and_run(tmp_path, "attention_rows_on_host", spliced_attention_rows_source())


def test_contractions_for_any_shape_in_bounds_and_correct_on_host(tmp_path):
    build_and_run(tmp_path, "gemm_any_on_host", spliced_gemm_any_source())


def build_and_run(tmp_path, name, source):
    cpp = tmp_path / (name + ".cpp")
    cpp.write_text(source)
    exe = tmp_path / name
    cmd = ["g++", "-O1", "-g", "-fsanitize=address,undefined", "-fno-sanitize-recover=all", "-static-libasan",
           "-static-libubsan", "-std=c++20", "-pthread", "-I", os.path.join(HERE, "host_emulation"),
           "-I", os.path.join(ROOT, "include"), str(cpp), "-o", str(exe)]
    r = subprocess.run(cmd, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-3000:]
    env = dict(os.environ, ASAN_OPTIONS="detect_leaks=0")
    r = subprocess.run([str(exe)], capture_output=True, text=True, env=env, timeout=600)
    assert r.returncode == 0 and r.stdout.strip().endswith("ok"), (r.stdout[-2000:], r.stderr[-3000:])


def rule(name, signature):
    """One function of a dispatch, from its signature to the brace that closes it."""
    src = open(os.path.join(CSRC, name)).read()
    i = src.index(signature)
    return src[i:src.index("\n}\n", i) + 3]


def ask_rules(tmp_path, questions):
    internal = open(os.path.join(CSRC, "aqt_internal.h")).read()
    shape = internal[internal.index("struct AttnShape {"):]
    shape = shape[:shape.index("};") + 2]
    enum = re.search(r"^enum class Tile .*$", open(os.path.join(CSRC, "gemm_any.hip")).read(), flags=re.M).group(0)
    rules = [enum, rule("gemm_any.hip", "Tile pick_tile("), rule("gemm_any.hip", "bool dense_fwd_rows_ok("), rule("block.hip", "int grid_cap("),
             rule("block.hip", "int layernorm_blocks("), "constexpr int kQf = 16;", rule("attention_few.hip", "bool attention_few_ok("), rule("attention_bwd.hip", "bool attention_bwd_few_ok(")]
    source = ('#include <stdint.h>\n#include <stdio.h>\n#include <string.h>\n#include "aqt.h"\nnamespace aqt {\n'
              'inline int64_t cdiv(int64_t a, int64_t b) { return (a + b - 1) / b; }\n' + shape + "\n" + "\n".join(rules) + "\n}\n" +
              open(os.path.join(HERE, "host_emulation", "rules_driver.cpp")).read())
    cpp, exe = tmp_path / "rules.cpp", tmp_path / "rules"
    cpp.write_text(source)
    r = subprocess.run(["g++", "-O1", "-std=c++17", "-I", os.path.join(ROOT, "include"), str(cpp), "-o", str(exe)], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-3000:]
    r = subprocess.run([str(exe)], input="\n".join(" ".join(str(v) for v in q) for q in questions), capture_output=True, text=True, timeout=60)
    return [int(v) for v in r.stdout.split()]


# utterances, frames, heads, head width, left, right -> whether 32 rows to a workgroup were measured to be the faster
BWD_FEW = [((25, 16, 4, 4, -1, -1), 0), ((62, 16, 4, 64, -1, -1), 0), ((100, 32, 2, 24, -1, -1), 0), ((1, 1, 1, 4, -1, -1), 0),
           ((50, 33, 2, 36, -1, -1), 1), ((8, 128, 4, 64, 23, 0), 1), ((2, 1000, 4, 64, -1, -1), 1), ((16, 128, 4, 64, -1, -1), 1),
           ((19, 128, 4, 64, -1, -1), 0), ((8, 288, 4, 64, -1, -1), 0), ((18, 401, 2, 4, -1, -1), 0), ((18, 401, 2, 24, -1, -1), 0),
           ((18, 401, 2, 64, -1, -1), 1), ((17, 417, 2, 32, -1, -1), 0), ((17, 417, 2, 48, -1, -1), 1), ((15, 512, 2, 24, -1, -1), 1),
           ((16, 480, 2, 16, -1, -1), 0), ((7, 1000, 2, 4, -1, -1), 1), ((16, 480, 2, 4, -1, 0), 1), ((18, 401, 2, 4, -1, 0), 0),
           ((7, 1000, 2, 24, 200, 200), 1), ((17, 420, 2, 4, 200, 200), 0), ((17, 420, 2, 4, 420, 420), 0), ((8, 1000, 4, 64, -1, -1), 0)]


# ... -> whether tiles of 16 queries were
FWD_FEW = [((6, 217, 4, 36, -1, -1), 1), ((8, 128, 8, 64, -1, -1), 1), ((8, 217, 8, 64, -1, -1), 0), ((31, 32, 4, 24, -1, -1), 1),
           ((50, 32, 4, 24, -1, -1), 0), ((37, 17, 4, 64, -1, -1), 0), ((50, 32, 4, 4, 23, 0), 0), ((33, 48, 4, 24, -1, -1), 1),
           ((25, 64, 4, 48, -1, -1), 0), ((25, 64, 4, 48, 23, 0), 1), ((25, 64, 4, 24, 63, 64), 0), ((25, 64, 4, 64, -1, -1), 1),
           ((25, 64, 4, 16, -1, -1), 1), ((100, 16, 4, 36, -1, -1), 1), ((100, 16, 4, 48, -1, -1), 0), ((100, 8, 4, 48, -1, -1), 1),
           ((1, 40, 8, 64, 23, 0), 1), ((25, 65, 4, 24, -1, -1), 1)]


# rows, fan-in, columns -> whether the product that makes its own codes was the faster
OWN_CODES = [((5000, 144, 144), 1), ((2600, 256, 256), 1), ((2000, 320, 320), 1), ((6000, 384, 96), 1), ((600, 400, 400), 1),
             ((1302, 512, 128), 1), ((40, 512, 512), 1), ((2600, 512, 128), 0), ((4000, 480, 120), 0), ((4000, 400, 100), 0),
             ((1302, 512, 512), 0), ((600, 512, 512), 0), ((800, 448, 448), 1), ((1200, 400, 400), 1), ((1580, 400, 400), 0), ((40, 516, 64), 0), ((40, 60, 64), 0), ((3000, 128, 512), 0)]


# rows, width, whether in pieces of 16 bytes -> workgroups of the normalisation's two passes, 2048 (8192 wavefronts) where even shares were slower
LN_BLOCKS = [((1, 512, 1), 1), ((8193, 512, 1), 1025), ((24577, 512, 1), 1537), ((10008, 1028, 1), 1251), ((10008, 2048, 1), 2048),
             ((24577, 1501, 0), 2048), ((24577, 257, 0), 2048), ((17000, 257, 0), 1417), ((9000, 1500, 1), 2048), ((40, 2048, 1), 10)]


def test_dispatch_rules_follow_the_measurements(tmp_path):
    cases = [(("attention_bwd_few",) + q, want) for q, want in BWD_FEW] + [(("attention_few",) + q, want) for q, want in FWD_FEW]
    cases += [(("own_codes",) + q, want) for q, want in OWN_CODES] + [(("layernorm_blocks",) + q, want) for q, want in LN_BLOCKS]
    got = ask_rules(tmp_path, [q for q, _ in cases])
    assert len(got) == len(cases)
    assert [(q, w) for (q, w), g in zip(cases, got) if g != w] == []
