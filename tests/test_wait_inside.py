"""Waits inside a workgroup of the kernels whose workgroups wait for each other: the rule (csrc/wait_inside.h) in simulated time, and that every such wait follows
it.  On the CPU."""
import os
import re
import subprocess

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_2410_12513_amd", "csrc")


def test_a_wait_inside_a_workgroup_outlasts_the_poll_it_depends_on(tmp_path):
    exe = str(tmp_path / "wait_inside_model")
    subprocess.run(["g++", "-std=c++17", "-O2", os.path.join(HERE, "wait_inside_model.cpp"), "-o", exe], check=True)
    res = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    assert res.returncode == 0 and res.stdout == "ok\n", res.stdout


def test_no_wait_of_the_batched_step_goes_on_without_what_it_waits_for():
    """A wait that ends gets its result looked at - the streaming wave's, whose code has no branch there, by the word that says so -, and none counts its own
    turns."""
    with open(os.path.join(CSRC, "batch_step.h")) as fh:
        code = re.sub(r"//.*", "", fh.read())
    body = code[code.index("k_empty_words("):]                              # (behind the waits' own definitions)
    assert not re.search(r"SK_SPIN_LIMIT|INSIDE_LIMIT|wait_inside|while \(bs_count", body)
    calls = [m.start() for m in re.finditer(r"\bbs_(?:poll|inside)\(", body)]
    assert len(calls) >= 8
    unlooked = [body[at:at + 24] for at in calls if not re.search(r"if \(!?$", body[body.rindex("\n", 0, at) + 1:at])]
    assert unlooked == ["bs_inside(link.bad, link"] and re.search(r"bs_count\(link\.bad\) == 0 && lane == 0\) __hip_atomic_fetch_add\(link\.done", body)


def test_only_polls_of_memory_have_the_shorter_limit():
    for name in sorted(os.listdir(CSRC)):
        with open(os.path.join(CSRC, name)) as fh:
            code = re.sub(r"//.*", "", fh.read())
        uses = [line for line in code.splitlines() if "SK_SPIN_LIMIT" in line]
        want = {"wait_inside.h": "constexpr unsigned SK_SPIN_LIMIT", "step_kernel.h": "((unsigned)e >> 1) - 1u : SK_SPIN_LIMIT"}.get(name)
        assert len(uses) == (want is not None) and all(want in line for line in uses), (name, uses)
