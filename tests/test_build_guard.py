"""The build refuses device functions so large that a branch within one may need a long branch."""
import shutil
import subprocess

import pytest

from paper_2306_03574_amd import build as b

HEAD = """
Symbol table '.symtab' contains 5 entries:
   Num:    Value          Size Type    Bind   Vis       Ndx Name
"""


def _row(n, size, kind, name):
    return f"     {n}: 0000000000001000 {size:5d} {kind:7} LOCAL  DEFAULT    7 {name}\n"


def test_functions_by_size():
    table = HEAD + _row(1, b.BRANCH_REACH - 4, "FUNC", "_Zshort") + _row(2, b.BRANCH_REACH, "FUNC", "_Zlong")
    table += _row(3, 1 << 20, "FUNC", "_Zkernel") + _row(4, 64, "OBJECT", "_Zkernel.kd") + _row(5, 99999, "FUNC", "_Zs")
    assert b.overlong_functions(table) == ["_Zlong"]
    assert b.overlong_functions(table.replace("_Zlong", "_Zshort").replace(str(b.BRANCH_REACH), "   12")) == []


def test_on_a_compiled_object(tmp_path):
    cc = b.hipcc()
    src, obj = tmp_path / "x.hip", tmp_path / "x.o"
    # one device function above the reach (a chain of distinct stores), one below, and a kernel
    src.write_text("""#include <hip/hip_runtime.h>
template <int N> __device__ __forceinline__ void chain(volatile int* p) {
  if constexpr (N == 1) { p[0] = 12345; } else { chain<N / 2>(p); chain<N - N / 2>(p); }
}
__device__ __attribute__((noinline)) void far_function(volatile int* p) { chain<16384>(p); }
__device__ __attribute__((noinline)) void near_function(volatile int* p) { chain<16>(p); }
__global__ void kernel(int* p) { far_function(p); near_function(p); }
""")
    subprocess.run([cc] + [f for f in b.HIPCC_FLAGS if f != "-shared"] + ["-c", str(src), "-o", str(obj)], check=True,
                   capture_output=True)
    names = b.overlong_functions(b.device_symbols(str(obj)))
    assert len(names) == 1 and "far_function" in names[0]
    with pytest.raises(RuntimeError, match="past the reach"):
        csrc = tmp_path / "csrc"
        csrc.mkdir()
        shutil.copy(src, csrc / "x.hip")
        with pytest.MonkeyPatch.context() as mp:
            mp.setattr(b, "SOURCES", ["x.hip"])
            b.build(csrc=str(csrc), lib=str(tmp_path / "x.so"))
