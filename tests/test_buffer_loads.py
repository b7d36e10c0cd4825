"""The kernels' range-checked loads, in the library as it is built.

A buffer load returns 0 past its descriptor's range only as far as the vector
and the immediate offset go; the scalar offset is added after the check.  So
every one has to carry 0 there, or the last, partly filled tile of a matrix
could read past col and val."""
import os
import re
import subprocess

from paper_1504_06474_amd import build

OBJDUMP = os.path.join(os.environ.get("ROCM_PATH", "/opt/rocm"), "llvm", "bin", "llvm-objdump")


def device_assembly(tmp_path):
    if not os.path.exists(build.LIB):
        build.build()
    lib = tmp_path / "libsss.so"
    lib.symlink_to(build.LIB)
    subprocess.run([OBJDUMP, "--offloading", str(lib)], cwd=tmp_path, check=True, capture_output=True)
    objects = sorted(p for p in tmp_path.iterdir() if p.name.endswith("gfx950"))
    assert objects
    return "\n".join(subprocess.run([OBJDUMP, "-d", "--mcpu=gfx950", str(p)], check=True, capture_output=True,
                                    text=True).stdout for p in objects)


def test_no_scalar_offset(tmp_path):
    loads = re.findall(r"^\s+(buffer_load_\S+ .*?)\s*//", device_assembly(tmp_path), re.M)
    assert len(loads) > 100
    # buffer_load_x  dst, vaddr, s[descriptor], soffset ...
    bad = [i for i in loads if re.search(r"s\[\d+:\d+\], (\S+)", i).group(1) != "0"]
    assert not bad, bad[:5]


RANGES = r"""
#include <cstdio>
#include <initializer_list>
#include "sss_internal.h"
int main() {
  for (unsigned size : {2u, 4u, 8u})
    for (unsigned count = 0; count <= 3000; ++count) {
      const unsigned r = value_range(count, size), end = count * size;
      if (r > end || r % 4 || r + (size == 2 && count % 2 ? 2 : 0) != end) return std::printf("%u x %u: %u\n", count, size, r), 1;
    }
}
"""


def test_ranges_end_with_the_values(tmp_path):
    """Never a byte past the last value, and every value but an odd last one of
    16 bits."""
    src, exe = tmp_path / "r.cpp", tmp_path / "r"
    src.write_text(RANGES)
    csrc = os.path.join(build.HERE, "csrc")
    subprocess.run(["g++", "-std=c++17", "-I", csrc, "-I", os.path.join(build.ROOT, "include"), str(src), "-o", str(exe)],
                   check=True)
    subprocess.run([str(exe)], check=True)
