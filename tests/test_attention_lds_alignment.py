"""The attention kernels change K buffers by an exclusive or of their LDS addresses with the tile's size: the array has to
start at a multiple of two tiles.  Checked on what the compiler is told (its intermediate form of the kernels)."""
import re
import subprocess

from paper_2603_06664_amd import build


def test_tile_buffers_are_aligned_to_two_tiles(tmp_path):
    out = str(tmp_path / "attention.ll")
    subprocess.run(["hipcc", *build.FLAGS, *build.SOURCE_FLAGS.get("attention.hip", []), "-S", "-emit-llvm", "--cuda-device-only",
                    build.os.path.join(build.CSRC, "attention.hip"), "-o", out], check=True, stdout=subprocess.DEVNULL,
                   stderr=subprocess.DEVNULL)
    with open(out) as f:
        arrays = re.findall(r"^@.*addrspace\(3\) global \[(\d+) x i8\].*align (\d+)", f.read(), re.M)
    assert len(arrays) == 8, arrays   # 2 work-group shapes x limited or not x folded or not
    for size, align in arrays:
        assert int(size) in (5 * 64 * 256, 5 * 128 * 256)   # two K tiles and three V tiles of 64 or 128 rows
        assert int(align) % (2 * int(size) // 5) == 0, (size, align)
