"""What the library's host code does with the buffers that results come back through, on a HIP
runtime that lives in host memory (fake_hip.cpp) and refuses what the test says."""
import os
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_2207_08207_amd", "csrc")


@pytest.fixture(scope="module")
def fake(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("fake") / "fake_hip")
    rocm = os.environ.get("ROCM_PATH", "/opt/rocm")
    subprocess.run(["g++", "-std=c++17", "-O1", "-g", "-w", "-D__HIP_PLATFORM_AMD__", "-D__align__(x)=",
                    "-DHIP_SYMBOL(x)=(&x)", f"-I{rocm}/include", f"-I{CSRC}", "-x", "c++",
                    os.path.join(HERE, "fake_hip.cpp"), "-o", exe, "-lpthread"], check=True)
    return exe


def run(exe, *args):
    r = subprocess.run([exe, *map(str, args)], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0 and r.stdout.strip() == "ok", r.stdout + r.stderr


def test_candidates_of_a_batch(fake):
    run(fake, "plain")


def test_a_refused_result_buffer_is_no_error(fake):
    """The candidates' pinned buffer is optional: the event is enqueued without it, and its results
    are copied from the device."""
    run(fake, "refused")


@pytest.mark.parametrize("scenario", ["unstaged", "unpooled"])
def test_results_without_a_pinned_buffer(scenario, fake):
    """The getters copy straight into the caller's arrays when no pinned buffer is to be had, and when
    the result is larger than any that the pool keeps."""
    run(fake, scenario)


def test_a_failed_event_outlives_its_stream(fake):
    run(fake, "failed")


def test_host_memory_of_held_events(fake):
    """Sized by the event, at most 64 MiB for all that are held, room for four PU200 events, none for more."""
    run(fake, "room")


def test_the_autotuner_skips_sites_without_a_shape(fake):
    run(fake, "tune")
