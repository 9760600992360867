"""Bookkeeping of whole calls without a GPU: the built library runs on a
stand-in for the HIP runtime (tests/host: host memory, kernels that do nothing,
streams whose work stays pending), which sees every allocation, wait and launch
that a call makes."""
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    if shutil.which("gcc") is None:
        pytest.skip("gcc not available")
    lib = os.path.join(ROOT, "paper_2111_07886_amd", "libpet_os.so")
    if not os.path.exists(lib):
        from paper_2111_07886_amd import build
        build.build()
    exe = str(tmp_path_factory.mktemp("host") / "calls")
    # -rdynamic: the library's HIP calls resolve to the program's
    subprocess.run(["gcc", "-O1", "-g", "-std=gnu11", "-Wall", "-rdynamic", "-I", os.path.join(ROOT, "include"),
                    os.path.join(HERE, "host", "calls.c"), os.path.join(HERE, "host", "hip_stub.c"), "-o", exe, lib,
                    "-Wl,-rpath," + os.path.dirname(lib), "-lpthread"], check=True, capture_output=True)
    return exe


def run(program, scenario):
    res = subprocess.run([program, scenario], capture_output=True, text=True, timeout=60)
    assert res.returncode == 0 and res.stdout.strip() == "ok", res.stdout + res.stderr


def test_a_failed_call_gives_back_scratch_in_order(program):
    """A call that runs out of memory gives back scratch that another stream's
    queued work still uses: the next call waits for it or takes other memory."""
    run(program, "failed_call")


def test_kept_memory_is_bounded_over_all_geometries(program):
    """At most 256 MiB per device stay with the library between calls, whatever
    the number of geometries; its own allocations get them when memory is out,
    and the last geometry's end frees them."""
    run(program, "memory_kept")


def test_streams_do_not_wait_for_each_other(program):
    """Back-projections on two streams, and whole calls on a third, take scratch
    that no other stream's queued work uses."""
    run(program, "streams")


def test_a_back_projection_stays_asynchronous(program):
    """A back-projection neither waits nor frees, whatever its scratch finds: 40
    streams at once, more than the kept blocks hold, and no memory left."""
    run(program, "asynchronous")


def test_a_back_projection_beside_a_capture(program):
    """A back-projection on one stream makes no call that ends the capture of
    another stream (global capture mode forbids allocations and event queries)."""
    run(program, "beside_a_capture")


def test_a_failed_batch_step_is_taken_up_again(program):
    """A launch that fails, at every place of two batched steps: the steps before
    it are counted, and running on updates each request once per step."""
    run(program, "failed_step")


def test_launches_of_images_with_many_rows(program):
    """Every launch for an image of 70001 rows, or for 8200 angles of 1101 bins, is
    within the limits of a grid."""
    run(program, "large_grids")


def test_the_autotuner_times_what_subiterations_use(program):
    """No trial launches for a 3D geometry whose subiterations go by quads."""
    run(program, "autotune")


def test_memory_for_the_sinogram_bin_by_bin_is_enough(program):
    """States, reconstructions, gradients and batches that have memory for the
    subset sinogram bin by bin, but not in the 3D projectors' own layout, run."""
    run(program, "memory_limits")
