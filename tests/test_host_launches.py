"""What the host runtime launches, on the CPU: the runtime sources are compiled
with the HIP calls and the kernel launchers replaced by recorders
(``tests/host``), so rules that no field value shows can be checked without a
GPU (and before anything runs on one)."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HOST = os.path.join(ROOT, "tests", "host")
ROCM = os.environ.get("ROCM_PATH", "/opt/rocm")


@pytest.fixture(scope="module")
def driver(tmp_path_factory):
    built = {}

    def run(name, check):
        if name not in built:
            exe = str(tmp_path_factory.mktemp("host") / name)
            cmd = ["g++", "-std=c++17", "-O1", "-g", "-fsanitize=address,undefined", "-fno-sanitize-recover=undefined",
                   "-D__HIP_PLATFORM_AMD__", "-isystem", os.path.join(ROCM, "include"), "-I",
                   os.path.join(ROOT, "include"), "-I", os.path.join(ROOT, "paper_2010_01847_amd", "csrc"), "-I", HOST,
                   os.path.join(HOST, name + ".cpp"), "-o", exe]
            r = subprocess.run(cmd, capture_output=True, text=True)
            assert r.returncode == 0, r.stderr[-4000:]
            built[name] = exe
        r = subprocess.run([built[name], check], capture_output=True, text=True, timeout=120)
        assert r.returncode == 0 and f"{check}: ok" in r.stdout, r.stdout + r.stderr

    return run


def test_streams_share_no_check_records(driver):
    """Two streams of one call, a lone check step before block or fused check
    launches among the calls: neither writes records the other uses."""
    driver("lattice_launches", "streams")


def test_strips_follow_the_steps_of_a_launch(driver):
    """Few-step launches of large 16-bit handles take strips of half the
    height, in short calls, after lbm_set_step_fusion and after lbm_autotune."""
    driver("lattice_launches", "strips")


def test_block_plans_by_shape(driver):
    """The block kernels take a handle's lattices where their windows fit them:
    not thin ones, and whole lattices where a handle holds many small ones."""
    driver("lattice_launches", "plans")


def test_few_steps_and_check_steps_of_block_handles(driver):
    """Which kernels take few steps, check steps and a readout's replay of
    handles in the block kernels."""
    driver("lattice_launches", "short_runs")


def test_new_handles_pin_no_memory_without_use(driver):
    """lbm_create pins host memory only for handles with many check records;
    lbm_last_check never allocates."""
    driver("lattice_launches", "pinned")


def test_z_ranges_are_searched_once(driver):
    """Step calls on boxes of many planes cost no search of z ranges."""
    driver("box_launches", "ranges")


def test_z_ranges_by_box(driver):
    """The planes per block that a new handle takes for two steps per launch."""
    driver("box_launches", "planes")


def test_forms_of_the_gpu_tests(driver):
    """The GPU tests of the block kernels run the forms they name."""
    driver("lattice_launches", "forms")


def test_boxes_of_the_gpu_tests_take_three_steps(driver):
    """The GPU tests of three steps per launch run them."""
    driver("box_launches", "triples")
