"""Which kernels the calls launch, and in what grids: tests/host/launch_trace.cpp runs the
library's entry points on the host and records the launches in place of making them."""
import os
import subprocess

import pytest

import paper_1704_08657_amd as d
from test_batch_plan import ROOT, build_and_run, needs_tools

pytestmark = [needs_tools,
              pytest.mark.skipif(not os.path.exists(d.LIB_PATH), reason="the library is not built")]
DTYPES = {"f32": d.DWT2_F32, "bf16": d.DWT2_BF16, "f16": d.DWT2_F16, "i32": d.DWT2_I32}


@pytest.fixture(scope="module")
def trace(tmp_path_factory):
    """trace(calls): for each call its status and its launches (kernel, work-groups, threads)."""
    exe = tmp_path_factory.mktemp("host") / "launch_trace"
    subprocess.run(["g++", "-O2", "-std=c++17", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include",
                    "-I" + os.path.join(ROOT, "include"), os.path.join(ROOT, "tests", "host", "launch_trace.cpp"),
                    "-rdynamic", "-ldl", "-o", str(exe)], check=True)
    names = {}
    for line in subprocess.run(["nm", "-C", d.LIB_PATH], capture_output=True, text=True, check=True).stdout.splitlines():
        f = line.split(" ", 2)
        if len(f) == 3 and f[0] and "_kernel" in f[2] and "device_stub" not in f[2]:
            names[int(f[0], 16)] = f[2].split("(dwt2::Level")[0].split("(dwt2::Pair")[0].split("(dwt2_image")[0]

    def run(calls):
        r = subprocess.run([str(exe), d.LIB_PATH], input="\n".join(calls) + "\n", capture_output=True, text=True,
                           timeout=300)
        assert r.returncode == 0, r.stderr
        out = []
        for line in r.stdout.splitlines():
            st, *launches = line.split()
            out.append((int(st), [(names[int(a, 16)], int(g), int(t)) for a, g, t in
                                  (x.split(":") for x in launches)]))
        assert len(out) == len(calls)
        return out
    return run


def planes(direction, wavelet, dtype, n, h, w, levels, flags=0):
    return f"planes {direction} {d.WAVELETS[wavelet]} {DTYPES[dtype]} {n} {h} {w} {levels} {flags}"


def test_split_of_a_plane_stack(tmp_path):
    r = build_and_run(tmp_path, "launch_limit_check")
    assert r.returncode == 0, r.stdout + r.stderr
    assert "bad 0" in r.stdout


@pytest.mark.parametrize("wavelet,dtype", [("cdf97", "f32"), ("cdf97", "bf16"), ("cdf53", "i32"), ("cdf53f", "f16"),
                                           ("dd137", "f32"), ("dd137", "bf16")])
def test_launches_stay_below_the_work_item_limit(trace, wavelet, dtype):
    """Stacks of 2^23 planes and more, and single narrow images of very many tiles: every
    launch is of fewer than 2^32 work-items."""
    shapes = [((1 << 23) - 1, 4, 4, 2), (1 << 23, 4, 4, 2), (9000000, 4, 4, 1), (9000000, 16, 8, 3), (40000000, 4, 4, 2),
              (70000000, 2, 2, 1), (3000000, 100, 4, 2), (1, 1 << 27, 2, 1), (1, 1 << 27, 3, 2), (1, 330000000, 3, 2),
              (1, 390000000, 3, 2), (1, 460000000, 2, 1)]
    calls = [planes(direction, wavelet, dtype, *s) for s in shapes for direction in ("fwd", "inv", "adj")
             if direction != "adj" or wavelet == "cdf97"]
    for call, (st, launches) in zip(calls, trace(calls)):
        assert st == 0 and launches, call
        for name, groups, threads in launches:
            assert groups * threads < 1 << 32, (call, name, groups, threads)


def batch(dtype, levels, count, *sizes, flags=0):
    return f"batch {DTYPES[dtype]} {levels} {flags} {count} " + " ".join(f"{h} {w}" for h, w in sizes)


def test_batched_launches_stay_below_the_work_item_limit(trace):
    """9 million small images: one launch a level where two levels of them are too many
    work-items for one; 17 million, too many either way, are refused before any launch."""
    calls = [batch("f32", 2, 9000000, (4, 4)), batch("bf16", 3, 4500000, (5, 7), (6, 9)), batch("f32", 1, 9000000, (2, 3)),
             batch("f32", 1, 9000000, (2, 3), flags=d.DWT2_FLAG_KERNEL(1))]
    for call, (st, launches) in zip(calls, trace(calls)):
        if call is calls[3]:                              # a configuration of 512 threads a tile
            assert (st, launches) == (-2, []), call
            continue
        assert st == 0 and len(launches) > 1, call
        for name, groups, threads in launches:
            assert groups * threads < 1 << 32, (call, name, groups, threads)
    (st, launches), = trace([batch("f16", 2, 17000000, (4, 4))])
    assert (st, launches) == (-2, [])


def test_low_planes_take_the_low_tile(trace):
    """Two levels of planes that one tile of either height covers: the lower one."""
    for dtype, t in (("f32", "float, 0"), ("bf16", "__hip_bfloat16, {}")):
        calls = [planes(direction, "cdf97", dtype, 65536, h, 16, 2) for direction in ("fwd", "inv", "adj") for h in (4, 16, 40)]
        for call, (st, launches) in zip(calls, trace(calls)):
            i = ["fwd", "inv", "adj"].index(call.split()[1])
            assert st == 0
            assert [x[0] for x in launches] == [f"void dwt2::kern::pair::pair_kernel<{i}, 0, {t.format(0 if i == 2 else 3)}, 8, 4, 2>"], call


# the shapes of the GPU tests that compare the default calls with one launch a level
PAIR_SHAPES = [(1, 40, 224, 3), (2, 41, 225, 2), (3, 83, 460, 5), (130, 64, 192, 3), (64, 66, 193, 3), (1, 1501, 1499, 3),
               (3, 1079, 2017, 3), (3, 1080, 2016, 2), (3, 1083, 2050, 5), (1, 4099, 8201, 3), (1, 8192, 4096, 2)]
TAPS4_SHAPES = [(1, 27, 247, 2), (1, 111, 495, 2), (1, 200, 1000, 5), (1, 2900, 2050, 2), (3, 333, 1211, 4)]


@pytest.mark.parametrize("dtype", ["f32", "bf16", "i32"])
def test_every_multi_level_tile_is_compared_on_the_gpu(trace, dtype):
    """Among the shapes of tests/test_gpu_pair.py each tile of each direction is launched."""
    wavelet = "cdf53" if dtype == "i32" else "cdf97"
    for i, direction in enumerate(("fwd", "inv", "adj")):
        if direction == "adj" and dtype == "i32":
            continue
        seen = {name.split(", ", 4)[4] for call in trace([planes(direction, wavelet, dtype, *s) for s in PAIR_SHAPES])
                for name, _, _ in call[1] if f"pair::pair_kernel<{i}, " in name}
        assert seen >= {"8, 4, 2>", "8, 6, 2>", "12, 4, 3>", "16, 4, 3>"}, (direction, seen)


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_every_four_tap_tile_is_compared_on_the_gpu(trace, dtype):
    """Among the shapes of tests/test_gpu_taps4.py: one level in both heights, two levels in
    48 block rows and, forward with 16-bit storage, 64."""
    for i, direction in enumerate(("fwd", "inv")):
        calls = [planes(direction, "dd137", dtype, *s) for s in TAPS4_SHAPES]
        calls += [planes(direction, "dd137", dtype, *s, flags=d.DWT2_FLAG_FUSED) for s in TAPS4_SHAPES]
        names = {name for call in trace(calls) for name, _, _ in call[1]}
        assert all(f"taps4::" in n and f"_kernel<{i}, " in n for n in names), names
        two = {n.split(", ", 3)[3] for n in names if "pair_kernel" in n}
        one = {n.split(", ", 4)[3:][0] + ", " + n.split(", ", 4)[4] for n in names if "taps4_kernel" in n}
        assert two >= ({"8, 6>", "16, 4>"} if (direction, dtype) == ("fwd", "bf16") else {"8, 6>"}), two
        assert one >= {"4, 4, 2, 2>", "4, 5, 2, 2>"}, one


@pytest.mark.parametrize("flags", [0, d.DWT2_FLAG_PERSISTENT])
def test_low_images_take_the_low_tile(trace, flags):
    """A batch whose images all fit the height of the lower one-level tile takes that one."""
    levels = 2 if flags else 1
    calls = [batch("f16", levels, 700, (4, 16), (h, 5), flags=flags) for h in (7, 24, 25, 300)]
    for h, (st, launches) in zip((7, 24, 25, 300), trace(calls)):
        assert st == 0 and len(launches) == 2
        name, _, threads = launches[1]
        assert ("<__half, 3, 4, 4, 2>" if h <= 24 else "<__half, 3, 4, 6, 2>") in name, (h, name)


@pytest.mark.parametrize("n,h,w,rows", [(1, 1024, 1024, 4), (1, 2048, 2048, 4), (1, 3000, 3000, 6), (1, 8192, 8192, 6),
                                        (512, 256, 256, 6)])
def test_persistent_launch_takes_the_tall_tile_for_large_calls(trace, n, h, w, rows):
    for levels in (2, 5):
        (st, launches), = trace([planes("fwd", "cdf97", "f32", n, h, w, levels, d.DWT2_FLAG_PERSISTENT)])
        assert st == 0 and f"persist_fwd_kernel<float, 0, 4, {rows}, 2>" in launches[1][0]
    (st, launches), = trace([planes("fwd", "cdf97", "f32", n, h, w, 2, d.DWT2_FLAG_PERSISTENT | d.DWT2_FLAG_KERNEL(1))])
    assert st == 0 and "persist_fwd_kernel<float, 0, 8, 4, 2>" in launches[1][0]
