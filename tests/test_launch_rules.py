"""Rules that choose launch shapes, on the host (CPU): the library's own inline
functions, compiled into a small program and compared with what they have to
give."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2507_01152_amd", "csrc")


def _run(tmp_path, name, body, headers=("sg_internal.h",)):
    src, exe = tmp_path / f"{name}.cpp", tmp_path / name
    src.write_text("".join(f'#include "{h}"\n' for h in headers) +
                   "#include <cstdio>\n#include <vector>\nusing namespace sg;\n" + body)
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wno-unknown-pragmas", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include",
                    "-I" + CSRC, "-I" + os.path.join(ROOT, "include"), str(src), "-o", str(exe)], check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stdout[-2000:] + r.stderr[-2000:]
    return r.stdout


def test_every_ray_item_has_a_block(tmp_path):
    """Each item is taken by one block, however few blocks a GPU keeps resident."""
    _run(tmp_path, "items", """
int main()
{
    for (int resident = 1; resident <= 200; ++resident)
        for (int n = 1; n <= 400; n += (n < 140 ? 1 : 37)) {
            const int blocks = ray_blocks(resident, n);
            if (blocks < 1 || blocks > n) return std::printf("%d resident, %d items: %d blocks\\n", resident, n, blocks), 1;
            std::vector<int> seen(n, 0), taken(kRayQueues, 0);
            for (int b = 0; b < blocks; ++b)
                for (int i = b; i < n; i = ray_item(b, blocks, taken[b % kRayQueues]++)) ++seen[i];
            for (int i = 0; i < n; ++i)
                if (seen[i] != 1) return std::printf("%d resident, %d items: item %d taken %d times\\n", resident, n, i, seen[i]), 1;
        }
    return 0;
}
""")
