"""Column groups of the matrix-core product (csrc/mm_split.h, host code), compiled on its own: the chosen splits of
measured shapes, and their bounds. Sweeps of the number of groups on an MI355X say which splits are fast."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CHUNK, ROWS, MAX_CPG = 1024, 256, 1024


@pytest.fixture(scope="module")
def split(tmp_path_factory):
    cxx = shutil.which("g++") or "/opt/rocm/bin/amdclang++"
    d = tmp_path_factory.mktemp("mm_split")
    src = d / "main.cpp"
    src.write_text('#include <stdio.h>\n#include "mm_split.h"\nint main() {\n  long long r, c;\n'
                   '  while (scanf("%lld %lld", &r, &c) == 2) {\n'
                   f'    ds_mm_split s = ds_mm_choose_split(256, r, (r + {ROWS - 1}) / {ROWS}, (c + {CHUNK - 1}) / {CHUNK}, {MAX_CPG}, 32);\n'
                   '    printf("%lld %lld\\n", (long long)s.cpg, (long long)s.groups);\n  }\n  return 0;\n}\n')
    subprocess.run([cxx, "-O1", "-std=c++17", "-I", os.path.join(ROOT, "paper_2506_22668_amd", "csrc"), str(src),
                    "-o", str(d / "main")], check=True)

    def run(shapes):
        text = "\n".join(f"{r} {c}" for r, c in shapes)
        out = subprocess.run([str(d / "main")], input=text, capture_output=True, text=True, check=True).stdout.split()
        return list(zip(map(int, out[0::2]), map(int, out[1::2])))
    return run


# (rows, columns): numbers of groups whose CGLS iteration took at most 1 % longer than that of the fastest
FAST = {
    (34267, 99981): (5, 7, 8, 11), (99981, 34267): (3, 4, 5),          # 428 MB, 100,000 pairs of 99,981 players
    (10280, 99981): (6, 10, 11), (99981, 10280): (1,),
    (9424, 300007): (11, 12, 13), (300007, 9424): (1,),
    (57572, 1000175): (9, 10, 11, 20, 26), (1000175, 57572): (1, 2),
    (32409, 200003): (4, 6, 8, 10), (200003, 32409): (2, 3, 4),
    (15121, 500009): (8, 16, 17, 20, 38), (500009, 15121): (1,),
    (18176, 50021): (7,), (50021, 18176): (2, 5),
    (7906, 20011): (7, 8, 9), (20011, 7906): (3,),
    (3425, 100428): (25, 33), (100428, 3425): (1,),
}


def test_measured_shapes_take_a_fast_split(split):
    got = split(FAST)
    for shape, (cpg, groups) in zip(FAST, got):
        assert groups in FAST[shape], (shape, groups)


def test_every_split_covers_the_columns(split):
    shapes = [(1, 1), (1, 1024), (255, 1025), (256, 4096), (257, 1 << 20), (131072, 4097), (131073, 2049),
              (1, (1 << 22) + 5), (500000, 1 << 21), (3, 10 ** 7)]
    for (rows, cols), (cpg, groups) in zip(shapes, split(shapes)):
        chunks = -(-cols // CHUNK)
        assert 1 <= cpg <= MAX_CPG and (groups - 1) * cpg < chunks <= groups * cpg, (rows, cols, cpg, groups)
