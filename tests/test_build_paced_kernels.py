"""The build of a source with paced kernels: every kernel that asks for it comes
out spaced, or the build says which did not; tools that are missing leave the
kernel as it is, with a warning."""
import re
import subprocess

import pytest

from paper_2107_07104_amd.csrc import build as B

SOURCE = """#include <hip/hip_runtime.h>
#define FIB_PACED(on)                                \\
  do {                                               \\
    if constexpr (on) asm volatile("; fib paced");   \\
  } while (0)
template <bool PACED>
__global__ __launch_bounds__(64) void k_small(float* p, float a) {
  FIB_PACED(PACED);
  float v[16];
#pragma unroll
  for (int i = 0; i < 16; ++i) v[i] = p[threadIdx.x + 64 * i];
#pragma unroll
  for (int k = 0; k < 8; ++k)
#pragma unroll
    for (int i = 0; i < 16; ++i) v[i] = fmaf(v[i], a, v[(i + 1) % 16]);
#pragma unroll
  for (int i = 0; i < 16; ++i) p[threadIdx.x + 64 * i] = v[i];
}
void launch(float* p) { hipLaunchKernelGGL((k_small<INSTANCE>), 1, 64, 0, 0, p, 0.5f); }
"""


def _source(tmp_path, instance):
    src = tmp_path / "small.hip"
    src.write_text(SOURCE.replace("INSTANCE", instance))
    return str(src), str(tmp_path / "small.o")


def test_the_kernels_of_the_library_that_are_paced():
    names = []
    for src in B.SOURCES:
        with open(f"{B.HERE}/{src}") as f:
            text = f.read()
        found = B._PACED.findall(text)
        # every use of the macro is at the head of a kernel that is found
        assert len(found) == len(re.findall(r"^ *FIB_PACED\(", text, re.M))
        names += found
    assert sorted(names) == ["k_react_stream", "k_run_hh", "k_run_hh_adapt", "k_run_st57_adapt",
                             "k_window_hh"]


def test_a_kernel_that_is_not_spaced_is_named():
    long = ["\tv_add_f32 v0, v0, v1"] * 60
    def fn(name, marked):
        return [f"_Z{len(name)}{name}Pf:", *([f"\t{B.MARK}"] if marked else []), *long,
                "\ts_endpgm", ".Lfunc_end0:"]
    src = "".join(f"__global__ void {k}(float* p) {{\n  FIB_PACED(true);\n}}\n"
                  for k in ("k_one", "k_other"))
    both, _ = B.pace("\n".join(fn("k_one", True) + fn("k_other", True)))
    assert B.unspaced(src, both) == []
    one, n = B.pace("\n".join(fn("k_one", True) + fn("k_other", False)))
    assert n == 1 and B.unspaced(src, one) == ["k_other"]


def test_compile_with_and_without_the_tools(tmp_path, monkeypatch):
    src, obj = _source(tmp_path, "true")
    B._compile(src, obj, [])
    code = subprocess.run([f"{B.llvm_dir()}/llvm-objdump", "--offloading", obj], check=True,
                          capture_output=True, text=True)
    assert B.ARCH in code.stdout + code.stderr
    monkeypatch.setattr(B, "llvm_dir", lambda: str(tmp_path / "none"))
    with pytest.warns(RuntimeWarning, match="without spaced"):
        B._compile(src, obj + "2", [])
    assert (tmp_path / "small.o2").exists()
    src, obj = _source(tmp_path, "false")
    with pytest.raises(RuntimeError, match="k_small"):
        B._compile(src, obj, [])
