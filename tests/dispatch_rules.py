"""Asks the library's own host code which kernel a call takes: tests/host_rules/rules.cpp includes the headers that hold the
rules and is built once per session (host code, no GPU), under UndefinedBehaviorSanitizer."""
import functools
import os
import subprocess
import tempfile

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@functools.lru_cache(maxsize=None)
def _exe():
    exe = os.path.join(tempfile.mkdtemp(prefix="tvm_rules_"), "rules")
    cmd = ["hipcc", "--offload-arch=gfx950", "-O1", "-std=c++17", "-x", "hip",
           "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops", "-Wno-unused-command-line-argument",
           "-Xarch_host", "-fsanitize=undefined", "-Xarch_host", "-fno-sanitize-recover=all",
           os.path.join(ROOT, "tests", "host_rules", "rules.cpp"), "-o", exe]
    r = subprocess.run(cmd, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-3000:]
    return exe


def ask(queries):
    """queries: list of tuples (name, integers...).  Returns a list of tuples of integers."""
    text = "".join(" ".join(str(x) for x in q) + "\n" for q in queries)
    r = subprocess.run([_exe()], input=text, capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stderr[-3000:]
    lines = r.stdout.splitlines()
    assert len(lines) == len(queries) and not any(l.startswith("?") for l in lines), lines[:5]
    return [tuple(int(x) for x in l.split()) for l in lines]
