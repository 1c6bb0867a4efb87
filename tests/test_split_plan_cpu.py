"""The token split's plan (plain host arithmetic) over shapes on both sides of every rule, compiled with g++."""
import os
import subprocess

from split_shapes import SPLIT, WHOLE

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_split_plan_covers_every_token_and_leaves_room(tmp_path):
    exe = str(tmp_path / "check_split")
    subprocess.check_call(["g++", "-std=c++17", "-O2", "-Wall", "-fsanitize=undefined", "-fno-sanitize-recover=all",
                           os.path.join(ROOT, "tests", "split_plan", "check_split.cpp"), "-o", exe])
    pinned = {**SPLIT, **{(B, T, H): (1, T) for B, T, H in WHOLE}}
    args = [str(n) for shape, plan in pinned.items() for n in (*shape, *plan)]
    out = subprocess.run([exe, *args], capture_output=True, text=True)
    assert out.returncode == 0 and out.stdout.startswith("ok"), out.stdout + out.stderr
