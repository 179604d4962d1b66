"""The order of decode steps whose workgroups wait for each other (csrc/step_order.h) against a model of streams and events, on the CPU: random programs of contexts
that come, go and share streams.  The model also runs steps without any order and has to find some that meet."""
import os
import subprocess

HERE = os.path.dirname(os.path.abspath(__file__))


def test_steps_that_must_not_meet_are_ordered(tmp_path):
    exe = str(tmp_path / "step_order_model")
    subprocess.run(["g++", "-std=c++17", "-O1", os.path.join(HERE, "step_order_model.cpp"), "-o", exe], check=True)
    res = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    assert res.returncode == 0 and res.stdout == "ok\n", res.stdout
