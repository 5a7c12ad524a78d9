"""The adjoint's workspace: the least size carries no room for stored forward
passes that the call does not use, a larger workspace is used up to its end and
no further."""
import os
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
SAN = os.path.join(HERE, "sanitize")
CSRC = os.path.join(ROOT, "paper_2202_00086_amd", "csrc")
HIPCC = "/opt/rocm/bin/hipcc"


@pytest.mark.parametrize("n", [64, 512, 1024, 2048])
def test_least_size_has_no_store(n):
    """split_above -1: the one-lane path's checkpoints and segments (320 slots of 48
    bytes per lane), 30 bytes per pixel of lists and gradients, and the head.  With
    split sweeps: the records and segment items on top."""
    from paper_2202_00086_amd import kerrtrace as K
    lanes = min((n * n + 255) // 256 * 256, 65536)
    base = 320 * 48 * lanes + 30 * n * n
    sizes = {}
    for split in (-1, 0):
        cam, _, _, _, integ = K.make_structs(nx=n, ny=n, split_above=split)
        sizes[split] = K.kt_adjoint_workspace_bytes(cam, integ)
    assert base < sizes[-1] < base + (1 << 16)
    split_room = 1672 * lanes + 384 * min(n * n, 8192)
    assert base + split_room < sizes[0] < base + split_room + (1 << 16)


def test_room_for_every_pass():
    from paper_2202_00086_amd import kerrtrace as K
    header = open(os.path.join(ROOT, "include", "kerrtrace.h")).read()
    assert f"#define KT_ADJOINT_ROOM_PER_PIXEL {K.ADJOINT_ROOM_PER_PIXEL}\n" in header
    assert "#define KT_ADJOINT_ROOM_MAX ((size_t)8 << 30)\n" in header and K.ADJOINT_ROOM_MAX == 8 << 30
    for n, split, want in ((512, 0, 10240 * 512 * 512), (2048, 0, 8 << 30), (512, -1, None), (16, 0, None), (0, 0, 0)):
        cam, _, _, _, integ = K.make_structs(nx=n, ny=max(n, 1), split_above=split)
        assert K.adjoint_room(cam, integ) == (K.kt_adjoint_workspace_bytes(cam, integ) if want is None else want)


@pytest.mark.slow
def test_larger_workspaces_under_address_sanitizer(tmp_path):
    exe = str(tmp_path / "adjoint_room")
    subprocess.run([HIPCC, "-x", "hip", "--offload-host-only", "-std=c++17", "-g", "-O1", "-fno-omit-frame-pointer",
                    "-Xarch_host", "-fsanitize=address", "-Xarch_host", "-fsanitize=undefined",
                    "-Xarch_host", "-fno-sanitize-recover=all", "-w",
                    "-I", os.path.join(ROOT, "include"), "-I", CSRC, "-o", exe,
                    os.path.join(SAN, "adjoint_room_driver.cpp"), os.path.join(SAN, "stub_launch.cpp"),
                    os.path.join(CSRC, "kt_api.cpp")], check=True, capture_output=True)
    env = dict(os.environ, ASAN_OPTIONS="detect_leaks=0:abort_on_error=0")
    p = subprocess.run([exe], capture_output=True, text=True, timeout=600, env=env)
    assert p.returncode == 0 and p.stdout.startswith("ok "), p.stdout[-2000:] + p.stderr[-4000:]
