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


# pixels, channels, classes: the tile measured fastest, or within 5 % of it (whole rounds of one and two blocks per
# compute unit, ragged second rounds, every width)
GEMM_TILES = [(32550, 128, 1, 128, 128), (35340, 128, 1, 128, 128), (65100, 128, 1, 128, 128), (25947, 128, 1, 128, 128),
              (14880, 512, 1, 128, 128), (11904, 512, 1, 128, 128), (14880, 136, 1, 128, 128), (32550, 256, 1, 128, 128),
              (56730, 72, 1, 128, 128), (131072, 128, 1, 128, 128), (131000, 1024, 1, 128, 128), (17670, 192, 1, 128, 64),
              (21390, 192, 1, 128, 64), (8928, 136, 1, 64, 64), (6944, 256, 1, 64, 64), (11904, 128, 1, 64, 64),
              (2976, 512, 1, 64, 64), (2976, 128, 4, 64, 64), (1488, 136, 1, 32, 64), (589, 136, 1, 32, 64), (63, 1024, 1, 32, 64),
              (1, 72, 1, 32, 64), (131072, 64, 1, 128, 64), (65100, 64, 1, 128, 64), (56730, 64, 1, 128, 64), (32550, 64, 1, 64, 64),
              (25947, 40, 1, 64, 64), (5000, 64, 1, 32, 64),
              (8137, 64, 4, 64, 64), (130200, 32, 1, 128, 32), (56730, 24, 1, 128, 32), (26000, 32, 1, 64, 32),
              (130200, 8, 1, 256, 16), (130200, 16, 1, 256, 16), (33000, 16, 1, 64, 16)]


def test_gemm_tiles(tmp_path):
    out = _run(tmp_path, "tiles", """
int main()
{
    const long c[][3] = {%s};
    for (auto& x : c) {
        const GemmTile t = gemm_tile(x[0], x[1], (int)x[2]);
        std::printf("%%d %%d\\n", t.bm, t.bn);
    }
    return 0;
}
""" % ", ".join("{%d, %d, %d}" % t[:3] for t in GEMM_TILES), ("conv_rules.h",))
    got = [tuple(map(int, l.split())) for l in out.split("\n") if l]
    assert got == [t[3:] for t in GEMM_TILES], [(t, g) for t, g in zip(GEMM_TILES, got) if g != t[3:]]


# forward (0) or data gradient (1), channels in and out, upsampled, images, output size: whether the halo kernel was
# faster than the GEMM (the lines of the rule aside, by 5 % or more)
HALO = [(0, 64, 64, 0, 256, 16, 16, 1), (0, 64, 64, 0, 64, 17, 17, 0), (0, 64, 64, 0, 72, 17, 17, 0), (0, 64, 64, 0, 64, 31, 31, 1),
        (0, 64, 64, 0, 72, 24, 24, 0), (0, 64, 64, 0, 130, 24, 24, 0), (0, 64, 64, 0, 26, 20, 68, 0), (0, 64, 64, 0, 525, 18, 30, 0),
        (0, 64, 64, 0, 255, 16, 16, 0), (0, 64, 64, 0, 4200, 16, 16, 1), (0, 64, 128, 0, 32, 20, 68, 0), (0, 64, 128, 0, 16, 64, 64, 1),
        (0, 128, 64, 0, 32, 20, 68, 0), (0, 128, 64, 0, 32, 40, 40, 0), (0, 128, 64, 0, 16, 50, 50, 1), (0, 128, 64, 0, 1008, 16, 16, 1),
        (0, 128, 64, 0, 1024, 16, 16, 0), (0, 128, 64, 0, 200, 18, 30, 0), (0, 128, 128, 0, 64, 17, 17, 0), (0, 128, 128, 0, 32, 40, 40, 0),
        (0, 128, 128, 0, 8, 100, 100, 0), (0, 128, 128, 0, 128, 16, 16, 1), (0, 128, 128, 0, 165, 16, 16, 0), (0, 128, 128, 0, 6, 96, 104, 1), (0, 128, 128, 0, 400, 24, 16, 0),
        (0, 128, 512, 0, 16, 48, 20, 0), (0, 64, 64, 1, 200, 18, 18, 0), (0, 64, 64, 1, 64, 32, 32, 1), (0, 128, 64, 1, 200, 18, 30, 0),
        (0, 128, 64, 1, 64, 32, 32, 1), (0, 256, 64, 1, 72, 18, 18, 0), (0, 256, 64, 1, 16, 50, 50, 1), (0, 256, 128, 1, 525, 18, 18, 0),
        (1, 64, 64, 0, 290, 16, 16, 1), (1, 128, 128, 0, 300, 16, 16, 1), (1, 128, 64, 0, 1024, 16, 16, 0), (1, 64, 128, 0, 100, 16, 16, 0)]


def test_halo_kernel_where_it_pays(tmp_path):
    out = _run(tmp_path, "halo", """
int main()
{
    const int c[][7] = {%s};
    for (auto& x : c) std::printf("%%d\\n", (int)halo_pays(x[0], x[1], x[2], x[3], x[4], x[5], x[6]));
    return 0;
}
""" % ", ".join("{%s}" % ", ".join(map(str, t[:7])) for t in HALO), ("conv_rules.h",))
    got = [int(l) for l in out.split()]
    assert got == [t[7] for t in HALO], [t for t, g in zip(HALO, got) if g != t[7]]


# frames, width, height, radius, resident PSF blocks per compute unit with 64 and 32 scanlines: the tile measured faster
# (64 where they are within 2 %)
PSF_TILES = [(1, 64, 128, 2, 2, 3, 64), (64, 128, 256, 4, 2, 3, 64), (256, 128, 256, 4, 2, 3, 64), (256, 65, 256, 2, 2, 3, 64),
             (256, 33, 256, 1, 2, 3, 64), (64, 32, 256, 1, 2, 3, 64), (256, 32, 64, 1, 2, 3, 64), (256, 24, 256, 1, 2, 3, 32),
             (256, 32, 256, 1, 2, 3, 32), (256, 1, 256, 1, 2, 3, 32), (64, 256, 256, 16, 1, 3, 32), (256, 256, 256, 16, 1, 3, 32),
             (16, 256, 256, 16, 1, 3, 64), (256, 200, 200, 24, 1, 2, 32), (16, 200, 200, 24, 1, 2, 64), (1, 200, 200, 24, 1, 2, 32),
             (256, 128, 200, 20, 1, 2, 64), (256, 128, 128, 31, 1, 2, 64), (64, 256, 256, 31, 1, 2, 64), (16, 64, 64, 31, 1, 2, 32),
             (1, 128, 128, 4, 0, 2, 32)]


def test_psf_tile_width(tmp_path):
    out = _run(tmp_path, "psf", """
namespace sg { int psf_grid(int, int, int) { return 0; } }
int main()
{
    const int c[][6] = {%s};
    for (auto& x : c) {
        Extent e;
        for (int k = 0; k < x[0]; ++k) e.add(x[1], x[2]);
        std::printf("%%d\\n", psf_tile(e, x[3], 256, [&](int tx) { return 256 * x[tx == 64 ? 4 : 5]; }));
    }
    return 0;
}
""" % ", ".join("{%s}" % ", ".join(map(str, t[:6])) for t in PSF_TILES), ("sg_host.h",))
    got = [int(l) for l in out.split()]
    assert got == [t[6] for t in PSF_TILES], [t for t, g in zip(PSF_TILES, got) if g != t[6]]


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
