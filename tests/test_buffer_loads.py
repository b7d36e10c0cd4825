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
