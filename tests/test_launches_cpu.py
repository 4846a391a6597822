"""What the built library launches, without a GPU (tests/launch_drive.cpp stands
in for the HIP runtime): which kernel a shape takes, and that its grid, block
and LDS are within the device's limits."""
import os
import subprocess

import pytest

from paper_2301_09266_amd import finc

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
LDS = 160 * 1024


@pytest.fixture(scope="module")
def drive(tmp_path_factory):
    if not os.path.exists(HIPCC):
        pytest.skip("hipcc not found")
    exe = str(tmp_path_factory.mktemp("drive") / "launch_drive")
    subprocess.run([HIPCC, "--offload-host-only", "-x", "c++", "-std=c++17", "-O1", "-rdynamic",
                    "-I", os.path.join(ROOT, "include"), "-I", "/opt/rocm/include",
                    "-D__HIP_PLATFORM_AMD__", os.path.join(ROOT, "tests", "launch_drive.cpp"),
                    "-ldl", "-o", exe], check=True)

    def run(calls):
        """[(op, want, B, C, H, W, k, corner)] -> [(rc, [(kernel, blocks, threads, lds)])]"""
        text = "".join(" ".join(map(str, c)) + "\n" for c in calls)
        r = subprocess.run([exe, finc.LIB_PATH], input=text, capture_output=True, text=True,
                           timeout=120)
        assert r.returncode == 0, r.stderr
        out = []
        for line in r.stdout.splitlines():
            rc, *ls = line.split(";")
            out.append((int(rc), [(n, int(b), int(t), int(s)) for n, b, t, s in
                                  (x.rsplit(",", 3) for x in ls)]))
        assert len(out) == len(calls)
        return out
    return run


def names(launches):
    return ["gemm" if "gemm_grad_kernel" in n else "fwd" if "11grad_kernel" in n else
            "dk" if "9dk_kernel" in n else "sum" if "dk_reduce" in n else n
            for n, _, _, _ in launches]


# rows so wide that the row block's LDS size passes 2^32 floats and more, where
# a 32-bit size would come out small: (C, k, width), one row of one image
WIDE = [(20, 7, 16519032), (20, 7, 16519126), (52, 3, 16519100)] + [
    (C, k, W) for C, k in ((20, 7), (52, 3), (64, 7), (33, 5), (64, 2))
    for m in (1, 2) for cp in [(C + 3) // 4 * 4]
    for W in range(max(1, m * 2**32 // ((1 + 2 * (k - 1)) * cp) - 160),
                   m * 2**32 // ((1 + 2 * (k - 1)) * cp) + 8, 7) if W < 2**24]


def test_wide_rows_are_refused():
    for C, k, W in WIDE:
        for kind in (finc.PLAN_LAYER, finc.PLAN_UNIT):
            assert finc.forward_plan(kind, 1, C, 1, W, k) == finc.EUNSUPPORTED, (kind, C, k, W)


def test_inverse_of_wide_rows_is_streamed_or_refused():
    """Such an image is not held in LDS: up to 16 channels the stream form takes
    the layer, else it is refused."""
    for C, k, H in ((48, 3, 1), (5, 3, 2), (12, 7, 1), (20, 5, 2), (64, 2, 1), (33, 7, 16)):
        cp, P = (C + 3) // 4 * 4, k - 1
        for m in (1, 2, 3):   # the layout's sizes just past m 2^32 floats
            last = (m * 2**32 - (H + 2 * P) * 2 * P * cp) // ((2 * H + 2 * P) * cp)
            for W in range(last - 40, last + 400, 9):
                if not 0 < W * H < 2**24:
                    continue
                p = finc.inverse_plan(finc.PLAN_LAYER, C, H, W, k)
                if C <= 16:
                    assert p[0]["streamed"], (C, k, H, W)
                else:
                    assert p == finc.EUNSUPPORTED, (C, k, H, W, p)


def test_backward_of_wide_rows_is_a_gemm(drive):
    """Where the forward's row blocks do not fit, dx is the implicit GEMM: also
    past the forward's own bound of 2^24 pixels an image."""
    shapes = [(1, C, 1, W, k) for C, k, W in WIDE]
    shapes += [(1, 1, 1, 82595513, 7), (1, 1, 1, 214748361, 3), (1, 2, 3, 1 << 24, 3)]
    for s, (rc, ls) in zip(shapes, drive([("backward", 1, *s, 0) for s in shapes])):
        assert rc == finc.OK and names(ls) == ["gemm"], (s, rc, ls)
    rc, ls = drive([("backward", 1, 64, 12, 32, 32, 3, 0)])[0]
    assert rc == finc.OK and names(ls) == ["fwd"]


@pytest.mark.parametrize("want", [1, 2, 3])
def test_backward_grids(drive, want):
    """Every launch of the backward is one the device takes: under 2^32 threads
    (2^24 images of a pixel included), LDS of a workgroup, no empty grid."""
    shapes = [(1 << 24, 1, 2, 2, 3), ((1 << 24) - 1, 1, 1, 1, 3), (1 << 26, 4, 1, 1, 1),
              (1 << 20, 3, 2, 2, 3), (1, 1, 1, 1, 1), (64, 48, 8, 8, 3), (2, 64, 40, 40, 7),
              (33, 23, 27, 19, 5), (1, 12, (1 << 24) + 5, 1, 2), (1, 1, (1 << 31) - 130, 1, 1),
              (1 << 24, 1, 3, 3, 3), ((1 << 24) + 7, 1, 8, 8, 3), (3, 5, 2, 1000, 4)]
    for s, (rc, ls) in zip(shapes, drive([("backward", want, *s, 3) for s in shapes])):
        assert rc == finc.OK and ls, (s, rc, ls)
        for n, blocks, threads, lds in ls:
            assert 0 < blocks * threads < 2**32 and lds <= LDS, (s, n, blocks, threads, lds)


def test_backward_of_small_images(drive):
    """Small images share dK's bands, a pixel's are a GEMM in dx, and no launch
    has more blocks than the chip holds at a time however many images there are."""
    shapes = [(4096, 12, 2, 2, 3), (96, 12, 4, 4, 3), (4096, 12, 1, 1, 3), (20000, 3, 4, 4, 3)]
    (_, a), (_, b), (_, c), (_, d) = drive([("backward", 2, *s, 0) for s in shapes])
    # dk_kernel<k, FORM, BIG>: 1 several images a band, 2 and less halo
    for ls, form in ((a, 2), (b, 1), (c, 2), (d, 1)):
        assert "9dk_kernelILi3ELi%dELb0E" % form in ls[0][0], ls
    (_, a), (_, b), (_, c), (_, d) = drive([("backward", 1, *s, 0) for s in shapes])
    assert names(a) == names(c) == ["gemm"] and names(b) == names(d) == ["fwd"]
    assert d[0][1] <= 1024


def test_unit_forward_instances(drive):
    """forward_kernel<PADW, ROWS, threads>: 512 threads and weights in memory order
    up to 256 blocks; beyond, memory order only for whole channel tiles or whole
    sectors a row, and not where four blocks a compute unit run."""
    shapes = [((64, 20, 8, 8, 3), "ELb1ELi512E"), ((800, 20, 4, 4, 3), "ELb0ELi256E"),
              ((300, 33, 6, 6, 3), "ELb0ELi256E"), ((300, 40, 6, 6, 3), "ELb0ELi256E"),
              ((300, 32, 4, 4, 3), "ELb1ELi256E"), ((300, 24, 8, 8, 3), "ELb1ELi256E"),
              ((1000, 24, 3, 3, 2), "ELb0ELi256E"), ((300, 44, 4, 4, 2), "ELb1ELi256E"),
              ((256, 12, 16, 16, 3), "ELb0ELi512E")]
    for (s, want), (rc, ls) in zip(shapes, drive([("unit", 0, *s, 0) for s, _ in shapes])):
        assert rc == finc.OK and "14forward_kernelILb1" + want in ls[0][0], (s, ls)


def test_step_network_launches(drive):
    """The network in one launch where its scratch holds the packed weights, else
    the split GEMMs; not split below 8 channels (fp32 instruction) and, layer by
    layer, above 512."""
    def run(B, C, H, hid):
        rc, ls = drive([("step", hid, B, C, H, H, 3, 0)])[0]
        assert rc == finc.OK and all(b * t < 2**32 and s <= LDS for _, b, t, s in ls)
        return " ".join(n for n, _, _, _ in ls)
    for case, one, split in (((100, 12, 16, 512), True, False), ((1, 12, 8, 512), False, True),
                             ((128, 12, 16, 8), True, False), ((128, 12, 16, 7), False, False),
                             ((64, 64, 4, 64), True, True), ((100, 12, 16, 513), False, True)):
        k = run(*case)
        assert ("coupling_net_kernel" in k) == one and ("split_gemm_kernel" in k) == split, (case, k)
