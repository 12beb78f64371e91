"""What the library's host code enqueues (launch shapes, waits, events, captures), without a GPU: the sources are compiled
for the host alone and linked with a stand-in for the HIP runtime, under AddressSanitizer and UBSan."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HERE = os.path.join(ROOT, "tests", "host_sanitize")
CSRC = os.path.join(ROOT, "paper_2602_21548_amd", "csrc")
ENV = dict(os.environ, ASAN_OPTIONS="detect_leaks=0:verify_asan_link_order=0", UBSAN_OPTIONS="halt_on_error=1")
ENV.pop("LD_PRELOAD", None)

CHECKS = ["move_shapes", "full_block_planes", "capped_odd_rows", "capped_full_blocks", "large_odd_layers", "full_block_lanes",
          "caller_syncs", "row_map_under_capture", "row_map_on_two_streams", "default_stream", "cached_arrays",
          "ceiling_policies", "planes_by_rows", "planes_lanes", "planes_layout", "row_map_split", "tile_divisor",
          "row_map_rule", "tile_order", "small_gathers", "odd_rows_order", "variants_order",
          "tile_rules", "flat_split", "full_blocks_alike"]


@pytest.fixture(scope="module")
def harness(tmp_path_factory):
    hipcc = "/opt/rocm/bin/hipcc" if os.path.exists("/opt/rocm/bin/hipcc") else shutil.which("hipcc")
    if not hipcc:
        pytest.skip("hipcc not found")
    out = tmp_path_factory.mktemp("launches")
    exe = str(out / "launch_harness")
    r = subprocess.run([hipcc, "--offload-arch=gfx950", "--offload-host-only", "-fuse-cuid=none", "-no-hip-rt", "-O1", "-g", "-std=c++17",
                        "-Xarch_host", "-fsanitize=address", "-Xarch_host", "-fsanitize=undefined", "-Wno-unused-command-line-argument",
                        "-Wno-unused-result", "-I" + os.path.join(ROOT, "include"), "-I" + CSRC,
                        os.path.join(HERE, "launch_harness.cpp"), "-o", exe], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-2000:]
    return exe


def test_every_check_is_run(harness):
    out = subprocess.run([harness], capture_output=True, text=True, env=ENV, timeout=60)
    assert out.stdout.split() == sorted(CHECKS)


@pytest.mark.parametrize("check", CHECKS)
def test_launches(harness, check):
    out = subprocess.run([harness, check], capture_output=True, text=True, env=ENV, timeout=300)
    assert out.returncode == 0 and out.stdout.strip() == "ok", (out.stdout + out.stderr)[-3000:]
