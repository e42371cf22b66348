"""The library's calls of the HIP runtime, recorded on the CPU by tests/launch_recorder.cpp (kernels do not run)."""
import os
import re
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def build_recorder(folder):
    from paper_2311_10090_amd import binding
    if not os.path.exists(binding.LIB_PATH):
        from paper_2311_10090_amd.build import build
        build(force=True)
    exe, lib = os.path.join(str(folder), "launch_recorder"), os.path.dirname(binding.LIB_PATH)
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-o", exe, os.path.join(ROOT, "tests", "launch_recorder.cpp"), "-L", lib, "-l:libmpe.so",
                           "-Wl,-rpath," + lib, "-L/opt/rocm/lib", "-Wl,-rpath-link,/opt/rocm/lib"])
    return exe


def record(exe, commands, units=256):
    """Per command (return code, lines it printed)."""
    r = subprocess.run([exe, str(units)], input="\n".join(commands) + "\n", capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stderr
    out, lines = [], []
    for line in r.stdout.splitlines():
        if line.startswith("rc "):
            out.append((int(line[3:]), lines))
            lines = []
        else:
            lines.append(line)
    assert len(out) == len(commands)
    return out


def launches(lines):
    """(kernel, blocks) of the launches among the lines."""
    return [(m[1], int(m[2])) for m in (re.match(r"launch (.*) grid (\d+) ", line) for line in lines) if m]
