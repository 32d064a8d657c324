"""The launches of the library's calls, recorded on the CPU (see
launch_recorder.c): batches and widths at the far end of what the calls
accept, where a grid of one workgroup per tile, row or group would pass the
2^32 threads of a launch."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
F32, BF16 = 0, 1


@pytest.fixture(scope="module")
def record(tmp_path_factory):
    """record(lines) -> [(status, [(grid x, y, z, threads of a workgroup)])]"""
    gcc = shutil.which("gcc")
    if gcc is None:
        pytest.skip("gcc not available")
    from paper_2603_04800_amd import _libpath
    libdir = os.path.dirname(_libpath.LIB)
    exe = str(tmp_path_factory.mktemp("rec") / "launch_recorder")
    r = subprocess.run([gcc, "-std=gnu99", "-Wall", "-Werror", "-rdynamic", "-I", os.path.join(ROOT, "include"),
                        os.path.join(ROOT, "tests", "launch_recorder.c"), "-o", exe, "-L", libdir, "-lmasq",
                        f"-Wl,-rpath,{libdir}", "-Wl,--allow-shlib-undefined"], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr

    def run(lines):
        r = subprocess.run([exe], input="\n".join(lines) + "\n", capture_output=True, text=True, timeout=120)
        assert r.returncode == 0, r.stderr
        out = []
        for line in r.stdout.splitlines():
            st, *la = line.split()
            out.append((int(st), [tuple(int(v) for v in e.split(",")) for e in la]))
        assert len(out) == len(lines)
        return out
    return run


@pytest.mark.parametrize("call", [
    # codes and u in one launch: up to where (T / 16 + T / 8) x 512 threads fit, past it two
    f"fused 44739200 16 16 16 2 {F32} {F32} {F32} 0", f"fused 44739300 16 16 16 2 {F32} {F32} {F32} 0",
    f"fused 67000000 16 16 128 2 {BF16} {BF16} {BF16} 0",
    # a row and a quarter of u rows a workgroup, after the split down-projection
    f"fused 13421772 4160 16 16 2 {BF16} {BF16} {BF16} 0", f"fused 13421773 4160 16 16 2 {BF16} {BF16} {BF16} 0",
    f"fused 16777215 8192 16 64 3 {F32} {BF16} {F32} 0",
    # fp64 products whose 64 x 32 tiles pass 2^24 workgroups: one row, and a C of many rows
    "dgemm 1 536870880 4", "dgemm 1 536870881 4", f"dgemm 1 {128 * (2 ** 24 - 1)} 1", "dgemm 8388480 4096 1",
    # small GEMM tiles past 2^24 workgroups: many rows of few channels, and few rows of many
    f"gemm 1073741824 16 16 {BF16} 0", f"gemm 1100000000 64 16 {BF16} 1", f"gemm 2147483647 16 16 {BF16} 0",
    f"gemm 33 16 1073741824 {BF16} 0", f"fused 33 16 1073741824 0 1 {BF16} {BF16} {BF16} 0",
    # the standalone compensation's last 32-row tile
    f"comp {16 * (2 ** 24 - 1)} 16 16 16 2 {BF16} {BF16} {BF16}",
])
def test_launches_stay_within_the_thread_limit(record, call):
    status, launches = record([call])[0]
    assert status == 0 and launches, (call, status, launches)


@pytest.mark.parametrize("T,K,N,w4,large", [
    # several rounds of 128 x 128 tiles against those of 256 x 256 (a persistent grid of 256 workgroups of 512
    # threads): packed weights of long rows and a short last round keep the smaller tiles
    (1000, 3584, 18944, 1, False), (800, 512, 18944, 1, False), (2300, 8192, 8192, 1, False),
    (2300, 512, 8192, 1, True), (6000, 3584, 3584, 1, True), (1280, 3584, 18944, 1, True),
    (3000, 18944, 8192, 1, True), (1600, 512, 18944, 0, True), (1600, 3584, 18944, 0, True),
    (2048, 3584, 3584, 0, False), (700, 3584, 8192, 0, False), (8192, 3584, 18944, 0, True),
])
def test_tile_shapes_of_several_rounds(record, T, K, N, w4, large):
    for status, launches in record([f"fused {T} {K} {N} 32 2 {BF16} {BF16} {BF16} {w4}", f"gemm {T} {K} {N} {BF16} {w4}"]):
        assert status == 0
        assert launches[-1] == (256, 1, 1, 512) if large else launches[-1][3] == 256, launches


def test_slow_compensation_keeps_the_small_tiles(record):
    """With fp32 factors or a rank past 64 the 256 x 256 kernel's compensation
    costs more than its rounds save."""
    (st, f32), (sb, bf16), (sr, r128) = record([f"fused 2343 768 13248 64 2 {F32} {F32} {F32} 0",
                                                f"fused 2343 768 13248 64 2 {F32} {BF16} {F32} 0",
                                                f"fused 2343 768 13248 128 2 {BF16} {BF16} {BF16} 0"])
    assert st == sb == sr == 0 and bf16[-1] == (256, 1, 1, 512)
    assert f32[-1] == r128[-1] == (1976, 1, 1, 256)
