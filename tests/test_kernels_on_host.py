"""What the kernels' correctness needs beside their arithmetic, checked without a GPU: the kernel sources are built for the
CPU and run thread by thread (tests/host_kernels/host_kernels.cpp).  Every access has to lie in the workspace or an array
of the call, every wave has to meet the same barriers, and between two barriers no wave may touch LDS that another one
writes.  What a workgroup reads of another one of the same launch has to be complete when the count shows that it has waited for."""
import os
import re
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HERE = os.path.join(ROOT, "tests", "host_kernels")
CSRC = os.path.join(ROOT, "paper_1907_03329_amd", "csrc")
CLANG = os.environ.get("HOST_CLANG", "/opt/rocm/llvm/bin/clang++")


def without_launches(text):
    """kernel<<<grid, threads, lds, st>>>(arguments) -> a call per thread (host_launch)"""
    def closing(at, opening, ending):
        depth = 0
        while True:
            depth += (text[at] in opening) - (text[at] in ending)
            if depth == 0:
                return at
            at += 1
    at = text.find("<<<")
    while at >= 0:
        start = re.search(r"\w+(<[^<>;]*>)?$", text[:at]).start()
        stop = text.index(">>>", at)
        depth, parts = 0, [""]
        for c in text[at + 3:stop]:
            depth += (c in "(") - (c in ")")
            if c == "," and depth == 0:
                parts.append("")
            else:
                parts[-1] += c
        end = closing(stop + 3, "(", ")")
        call = f"host_launch({parts[0]}, {parts[1]}, {parts[2]}, [&] {{ {text[start:at]}{text[stop + 3:end + 1]}; }})"
        text = text[:start] + call + text[end + 1:]
        at = text.find("<<<", start + len(call))
    return text


PARTS = ["lstm_backward_kernels", "lstm_backward_large_kernels", "lstm_forward_kernels", "lstm_forward_residual_kernels",
         "lstm_narrow_kernels", "lstm_narrow_fwd_residual_kernels", "lstm_narrow_bwd_kernels", "lstm_narrow_bwd_split_kernels",
         "lstm_together_kernels", "lstm_together_wide_kernels", "lstm_together_forecast_kernels", "lstm_together_reverse_kernels", "lstm_kernels", "es_kernels", "head_kernels"]

MOST_LOOKS = 64


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    """The kernel sources with what has no meaning on a CPU replaced: launches, LDS whose size the launch gives, the barrier in
    inline assembly, empty asm statements that hold the device compiler back, and the address space of an LDS pointer.  A wait
    for another workgroup is given up sooner."""
    d = str(tmp_path_factory.mktemp("host_kernels"))
    shutil.copytree(HERE, d, dirs_exist_ok=True)
    for name in os.listdir(CSRC):
        if not name.startswith(("lstm_", "es_kernels", "head_kernels", "three_term", "esrnn_internal", "device_utils", "plan")):
            continue
        text = without_launches(open(os.path.join(CSRC, name)).read())
        text = re.sub(r"extern __shared__ (__align__\(16\) )?float (\w+)\[\];", r"float *\2 = host_dynamic_lds;", text)
        text = re.sub(r'asm volatile\("s_waitcnt lgkmcnt\(0\)\\n\\ts_barrier"[^;]*;', "host_barrier();", text)
        text = re.sub(r'asm( volatile)?\(""[^;]*;', ";", text)
        assert "asm" not in re.sub(r"//.*", "", text) and "extern __shared__" not in text, name
        text = text.replace("__attribute__((address_space(3)))", "")
        if name == "lstm_together.h":
            text, found = re.subn(r"kMostLooks = 1 << \d+", f"kMostLooks = {MOST_LOOKS}", text)
            assert found == 1
            text = text.replace("__ballot(", "host_ballot(")
        open(os.path.join(d, name), "w").write(text)
    common = [CLANG, "-std=c++17", "-O1", "-w", f"-DHOST_MOST_LOOKS={MOST_LOOKS}", "-I", d, "-I", os.path.join(ROOT, "include")]
    trace = ["-fsanitize-coverage=edge,trace-loads,trace-stores"]
    parts = [(f"{part}.o", "kernels.cpp", trace + [f'-DPART="{part}.hip"']) for part in PARTS]
    parts += [("plan.o", "plan.cpp", []), ("main.o", "host_kernels.cpp", [])]
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


@pytest.mark.parametrize("narrow", ["", "100000"])
@pytest.mark.parametrize("series", [1, 40, 256, 500, 1024, 1500])
def test_twelve_wave_workgroups_have_one_class_each(program, series, narrow):
    env = {k: v for k, v in os.environ.items() if k != "ESRNN_NARROW_BELOW"}
    for hidden, T in ((40, 12), (40, 60), (64, 60)):
        for dilations in ((1, 2, 3), (5, 16, 60), (255, 256, 700)):
            out = subprocess.run([program, "plan", str(series), str(T), "4", "3", str(hidden), "0", "all"] + [str(d) for d in dilations],
                                 env=dict(env, ESRNN_NARROW_BELOW=narrow) if narrow else env, capture_output=True, text=True, check=True).stdout
            for d, found in zip(dilations, re.findall(r"dilation \d+ narrow \d (\d) chains \d+ (\d+)", out), strict=True):
                four_series, chains = (int(v) for v in found)
                if four_series and 4 * -(-series // 16) * chains <= 256:
                    assert chains == min(d, T - 6)


def run_step(program, narrow, *args, how="step"):
    r = subprocess.run([program, how] + [str(a) for a in args], env=dict(os.environ, ESRNN_NARROW_BELOW=str(narrow)),
                       capture_output=True, text=True)
    return r.returncode, r.stdout.strip()


# 4-series kernels: chains around a group of four positions and two, tiles of few positions, and the output stage and
# everything else of a step beside them
@pytest.mark.parametrize("hidden,window", SHAPES)
def test_waves_of_the_4_series_kernels_are_ordered(program, hidden, window):
    T = window + 3 + 7
    assert run_step(program, 100000, 64, T, window, 3, hidden, min(T, 4), 0, 0, T, 1, 4) == (0, "ok")
    T = window + 3 + 16
    assert run_step(program, 100000, 128, T, window, 3, hidden, min(T, 4), 0, 0.1, f"{T},{window + 4}", 1) == (0, "ok")


@pytest.mark.parametrize("positions", [1, 2, 3, 4, 5, 7, 9, 16])
def test_chains_of_every_length(program, positions):
    T = 4 + 3 + positions - 1
    assert run_step(program, 100000, 64, T, 4, 3, 32, 4, 0, 0, T, 1, 2) == (0, "ok")


# 64 groups of four series have eight chains for twelve classes; past 256 workgroups the reverse kernel has four waves
@pytest.mark.parametrize("hidden,series,positions,dilations", [(8, 256, 14, (12, 3)), (40, 128, 34, (16,)), (64, 128, 20, (16,))])
def test_several_chains_a_workgroup(program, hidden, series, positions, dilations):
    window = 64 if hidden == 64 else 4
    T = window + 3 + positions - 1
    assert run_step(program, 100000, series, T, window, 3, hidden, 4, 0, 0, f"{T},{window + 9}", *dilations) == (0, "ok")


@pytest.mark.parametrize("hidden,H", [(8, 1), (8, 64), (32, 17), (40, 8), (40, 48), (50, 18), (50, 40), (64, 33), (64, 64)])
def test_waves_of_the_output_stage_are_ordered(program, hidden, H):
    T = 20 + H + 9 if hidden > 8 else 8 + H + 9
    assert run_step(program, 0, 64, T, T - H - 9, H, hidden, 4, 0, 0, T, 1) == (0, "ok")


# recursions: one, two, four and eight steps a group, and the kernel for long periods at its limit; lengths of one step, of
# no multiple of a chunk, and of none that a window fits into
@pytest.mark.parametrize("m1,m2", [(0, 0), (1, 0), (1, 1), (2, 3), (4, 7), (9, 12), (23, 0), (24, 0), (25, 24), (24, 37), (60, 0), (24, 23)])
def test_waves_of_the_recursions_are_ordered(program, m1, m2):
    for lengths in ("61,1", "60,48", "7,25"):
        assert run_step(program, 0, 128, 61, 4, 3, 8, m1, m2, 0, lengths, 1) == (0, "ok")


def test_waves_of_the_recursions_with_the_largest_rings(program):
    assert run_step(program, 0, 64, 305, 4, 3, 8, 300, 148, 0, "303", 1) == (0, "ok")


# layers of one launch: 4-series layers only, and a 16-series layer behind one (here from 20 workgroups on)
@pytest.mark.parametrize("hidden,window", SHAPES)
def test_waves_of_layers_in_one_launch_are_ordered(program, hidden, window):
    T = window + 3 + 17
    for lam, dilations, together in ((0.1, (1, 2), "2 2"), (0, (1, 8), "2 0")):
        out = subprocess.run([program, "plan"] + [str(a) for a in (64, T, window, 3, hidden, lam, "all") + dilations],
                             env=dict(os.environ, ESRNN_NARROW_BELOW="20"), capture_output=True, text=True, check=True).stdout
        assert f"together {together}" in out
        assert run_step(program, 20, 64, T, window, 3, hidden, min(T, 4), 0, lam, f"{T},{window + 9}", *dilations) == (0, "ok")


# chains around a group of four positions, and of one position (a horizon whose outputs hold the words all the same)
@pytest.mark.parametrize("positions", [1, 2, 3, 4, 5, 8, 9, 10])
def test_chains_of_every_length_in_one_launch(program, positions):
    T = 4 + 24 + positions - 1
    for dilations in ((1, 2), (2, 1)) if positions > 1 else ((1, 1),):
        out = subprocess.run([program, "plan"] + [str(a) for a in (64, T, 4, 24, 40, 0, "all") + dilations], capture_output=True, text=True,
                             check=True).stdout
        assert "together 2 2" in out
        assert run_step(program, 100000, 64, T, 4, 24, 40, 4, 0, 0, T, *dilations) == (0, "ok")


# what a bf16 pair of packed operands looks like as a ticket: its top bit is set; and as a count: it never comes
@pytest.mark.parametrize("hidden,narrow,dilation", [(8, 100000, 2), (8, 20, 8), (40, 100000, 2), (50, 20, 8)])
def test_places_and_waits_end_whatever_the_words(program, hidden, narrow, dilation):
    T = 12 + 3 + 9
    assert run_step(program, narrow, 64, T, 12 if hidden > 8 else 8, 3, hidden, 4, 0, 0, T, 1, dilation, how="uncleared") == (0, "ok")
