"""What a kernel asks for of its argument block before it needs it (warm_kernargs, csrc/device_math.h) is there: every line of the
explicit arguments and nothing behind them.  Compiled for gfx950, no GPU is touched."""
import glob
import os
import re
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2307_07649_amd", "csrc")
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
FLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops"]
# arguments of a kernel: bytes of a struct of doubles, and whether an int (and its padding) goes before it
KERNELS = [(136, False), (192, False), (184, True), (264, False), (312, False), (352, False), (384, False), (456, False), (512, False),
           (776, False), (792, False), (832, False)]


def listing(tmp_path):
    src = '#include "tgnn_internal.h"\n#include "device_math.h"\nusing namespace tgnn;\ntemplate <int N> struct Args { double v[N / 8]; };\n'
    for i, (n, lead) in enumerate(KERNELS):
        lead_arg, lead_name = ("int x, ", "x, ") if lead else ("", "")
        src += f'extern "C" __global__ void k{i}({lead_arg}Args<{n}> a) {{ warm_kernargs({lead_name}a); }}\n'
    src += 'extern "C" __global__ void grid(Args<512> a) { warm_kernargs_and_grid(a); }\n'
    (tmp_path / "k.hip").write_text(src)
    subprocess.run([HIPCC, *FLAGS, "-I", CSRC, "--cuda-device-only", "-S", str(tmp_path / "k.hip"), "-o", str(tmp_path / "k.s")], check=True)
    return (tmp_path / "k.s").read_text()


def test_lines_are_those_of_the_arguments(tmp_path):
    text = listing(tmp_path)
    for name, n in [(f"k{i}", n + (8 if lead else 0)) for i, (n, lead) in enumerate(KERNELS)] + [("grid", 512)]:
        body = re.search(rf"^{name}:.*?s_endpgm", text, flags=re.S | re.M).group(0)
        at = [(m.group(1), int(m.group(2), 16)) for m in re.finditer(r"s_load_dword s\d+, (s\[\d+:\d+\]), (0x[0-9a-f]+)", body)]
        if name == "grid":   # the word behind the arguments, through a pointer of its own
            assert at[-1][1] == 0 and at[-1][0] != at[0][0]
            at = at[:-1]
        assert [o for _, o in at] == [64 * i for i in range((n + 63) // 64)] and at[-1][1] + 4 <= n, (name, at)
        size = int(re.search(rf"\.kernarg_segment_size:\s*(\d+)(?:(?!\.kernarg_segment_size).)*?\.name:\s*{name}\n", text, flags=re.S).group(1))
        assert size >= (n + 4 if name == "grid" else n)


@pytest.mark.parametrize("path", sorted(glob.glob(os.path.join(CSRC, "*.hip"))), ids=os.path.basename)
def test_calls_name_the_kernels_parameters(path):
    text = open(path).read()
    calls = [m.start() for m in re.finditer(r"\bwarm_kernargs\w*(?=[(<])", text)]
    for at in calls:
        head = text.rindex("__global__", 0, at)
        params = re.search(r"void (\w+)\(([^{]*)\)\s*\{", text[head:at], flags=re.S)
        names = [re.search(r"(\w+)\s*$", p).group(1) for p in params.group(2).split(",")]
        call = re.match(r"warm_kernargs(?:_and_grid)?\(([^)]*)\)", text[at:])
        assert call is not None and [a.strip() for a in call.group(1).split(",")] == names, (params.group(1), text[at:at + 60])
