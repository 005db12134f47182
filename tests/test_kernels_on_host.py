"""What the 16-series LSTM kernels' correctness needs beside their arithmetic, checked without a GPU: the kernel sources
are built for the CPU and run thread by thread (tests/host_kernels/host_kernels.cpp).  Every global access has to lie in
the workspace, every wave has to meet the same barriers, and between two barriers no wave may touch LDS that another one
writes."""
import os
import re
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HERE = os.path.join(ROOT, "tests", "host_kernels")
CSRC = os.path.join(ROOT, "paper_1907_03329_amd", "csrc")
CLANG = os.environ.get("HOST_CLANG", "/opt/rocm/llvm/bin/clang++")


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    """The kernel sources with what has no meaning on a CPU replaced: launches, the barrier in inline assembly, empty asm
    statements that hold the device compiler back, and the address space of an LDS pointer."""
    d = str(tmp_path_factory.mktemp("host_kernels"))
    shutil.copytree(HERE, d, dirs_exist_ok=True)
    for name in os.listdir(CSRC):
        if not name.startswith(("lstm_backward", "lstm_forward", "three_term", "esrnn_internal", "device_utils", "plan")):
            continue
        text = open(os.path.join(CSRC, name)).read()
        text = re.sub(r"(\w+<[^<>;]*>)<<<(.*?), 0, st>>>\(a\)",
                      r"host_launch([](const void *p) { \1(*static_cast<const std::decay_t<decltype(a)> *>(p)); }, &a, \2)", text)
        text = re.sub(r'asm volatile\("s_waitcnt lgkmcnt\(0\)\\n\\ts_barrier"[^;]*;', "host_barrier();", text)
        text = re.sub(r'asm( volatile)?\(""[^;]*;', ";", text)
        assert "asm" not in re.sub(r"//.*", "", text), name
        text = text.replace("__attribute__((address_space(3)))", "")
        open(os.path.join(d, name), "w").write(text)
    common = [CLANG, "-std=c++17", "-O1", "-w", "-I", d, "-I", os.path.join(ROOT, "include")]
    trace = ["-fsanitize-coverage=edge,trace-loads,trace-stores"]
    parts = [("reverse.o", "kernels.cpp", trace + ["-DREVERSE"]), ("forward.o", "kernels.cpp", trace), ("plan.o", "plan.cpp", []),
             ("main.o", "host_kernels.cpp", [])]
    jobs = [subprocess.Popen(common + extra + ["-c", os.path.join(d, src), "-o", os.path.join(d, obj)]) for obj, src, extra in parts]
    assert not any([j.wait() for j in jobs])
    out = os.path.join(d, "host_kernels")
    subprocess.run([CLANG, "-o", out] + [os.path.join(d, obj) for obj, _, _ in parts], check=True)
    return out


def run(program, *args):
    env = dict(os.environ, ESRNN_NARROW_BELOW="0")
    r = subprocess.run([program] + [str(a) for a in args], env=env, capture_output=True, text=True)
    return r.returncode, r.stdout.strip()


# (hidden, input window): every instantiated shape
SHAPES = [(8, 4), (8, 8), (32, 6), (32, 12), (32, 30), (40, 4), (40, 12), (40, 23), (40, 30), (40, 40), (50, 12), (50, 18), (50, 50), (64, 64)]


@pytest.mark.parametrize("hidden,window", SHAPES)
def test_waves_of_a_workgroup_are_ordered(program, hidden, window):
    # 40 series: tiles of all positions, half of them, none; chains of several positions and of one
    assert run(program, 40, window + 3 + 6, window, 3, hidden, 0, "all", 1, 4) == (0, "ok")
    assert run(program, 40, window + 3 + 3, window, 3, hidden, 0.1, "all", 2, 1) == (0, "ok")


@pytest.mark.parametrize("dilation", [30, 31, 715827883, 1 << 30, (1 << 31) - 1])
def test_dilations_past_the_last_position_stay_in_the_workspace(program, dilation):
    # 31 positions: from 31 on every position is a chain of its own
    assert run(program, 20, 45, 12, 3, 40, 0, "all", dilation, 2, dilation) == (0, "ok")


def chosen(program, hidden, series, dilation):
    """Per layer: 1 where the 4-series kernel was chosen, forward and reverse."""
    env = {k: v for k, v in os.environ.items() if k != "ESRNN_NARROW_BELOW"}
    out = subprocess.run([program, "plan", str(series), "60", "4", "3", str(hidden), "0", "all", str(dilation)], env=env,
                         capture_output=True, text=True, check=True).stdout
    return [tuple(int(v) for v in re.findall(r"narrow (\d) (\d)", line)[0]) for line in out.splitlines() if line.startswith("layer")]


# workgroups of the 16-series grid: series / 16 times the dilation
@pytest.mark.parametrize("series,dilation", [(16 * 64, 1), (16 * 65, 1), (16 * 32, 4), (16 * 159, 1), (16 * 160, 1), (16 * 40, 4)])
def test_kernel_kind_follows_the_measured_limits(program, series, dilation):
    groups = series // 16 * dilation
    for hidden in (8, 30, 40, 52):
        assert chosen(program, hidden, series, dilation) == [(int(groups < 65), int(groups < 65))]
    # the fp32 reverse kernel of the largest hidden sizes is slower than the 4-series one up to 159 workgroups
    for hidden in (53, 64):
        assert chosen(program, hidden, series, dilation) == [(int(groups < 65), int(groups < 160))]
