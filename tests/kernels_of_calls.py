"""Which kernel a forward call runs on, without a GPU (tests/host/kernels_of_calls.cpp, compiled with hipcc against the built library)."""
import re
import shutil
import subprocess
from pathlib import Path

from paper_1805_12549_amd import binding as B

ROOT = Path(__file__).resolve().parent.parent
LIB = ROOT / "paper_1805_12549_amd" / "libcg_conv.so"


def build(folder):
    """The driver's path, or None without hipcc or the library."""
    hipcc = "/opt/rocm/bin/hipcc" if Path("/opt/rocm/bin/hipcc").exists() else shutil.which("hipcc")
    if hipcc is None or not LIB.exists():
        return None
    exe = Path(folder) / "kernels_of_calls"
    r = subprocess.run([hipcc, "--offload-arch=gfx950", "-O1", "-std=c++17", "-Wall", "-rdynamic", "-I", str(ROOT / "include"),
                        "-I", str(LIB.parent / "csrc"), str(ROOT / "tests" / "host" / "kernels_of_calls.cpp"), "-L", str(LIB.parent), "-lcg_conv", "-Wl,-rpath," + str(LIB.parent),
                        "-o", str(exe)], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stderr[-3000:]
    return exe


def layer(in_dtype, n, h, w, c_in, c_out, *, c_base=None, k=3, stride=1, pad=None, groups=0, shuffle=False, out_dtype=None, epilogue=0,
          variant=B.CG_VARIANT_AUTO, n_max=None, rq_shift=0):
    """A line of the driver's input; c_base None: a dense layer."""
    out = {B.CG_I8: B.CG_I32}.get(in_dtype, B.CG_F32) if out_dtype is None else out_dtype
    return (in_dtype, out, n_max or n, n, h, w, c_in, c_out, c_in if c_base is None else c_base, k, stride, k // 2 if pad is None else pad, groups,
            int(shuffle), epilogue, variant, rq_shift)


def ask(exe, layers):
    """(kernel, template arguments, threads to a workgroup, types of its arguments) of each layer's first launch.  (Small-tile kernels of the same template
    arguments differ in the last: UniformArgs where every K step lies inside one tap, else DirectArgs.)"""
    text = "\n".join(" ".join(str(v) for v in line) for line in layers) + "\n"
    r = subprocess.run([str(exe)], input=text, capture_output=True, text=True, timeout=120)
    lines = r.stdout.splitlines()
    assert r.returncode == 0 and len(lines) == len(layers), r.stderr[-2000:]
    return [_launch(line) for line in lines]


def _launch(line):
    m = re.search(r"(\w+)(?:<([^()]*)>)?\(([^()]*)\) (\d+)$", line.replace("(anonymous namespace)", "anonymous"))
    assert m, line
    names = lambda text: tuple(a.strip().split("::")[-1] for a in text.split(","))
    return m.group(1), names(m.group(2) or ""), int(m.group(4)), names(m.group(3))


def lines(exe, mode, calls):
    """The default line for each call, in one of its modes."""
    text = "\n".join(" ".join(str(v) for v in call) for call in calls) + "\n"
    r = subprocess.run([str(exe), mode], input=text, capture_output=True, text=True, timeout=120)
    said = r.stdout.splitlines()
    assert r.returncode == 0 and len(said) == len(calls), r.stderr[-2000:]
    return said


def beside(exe, calls):
    """The launches of cg_conv_call_beside for layers (n, h, w, c_in, c_out, c_base, kernel, stride, channels of the 1x1, groups): each as `ask` gives it, and its
    workgroups."""
    out = []
    for line in lines(exe, "beside", calls):
        assert line.endswith(";"), line
        out.append([_launch(text.rsplit(" ", 1)[0]) + (int(text.rsplit(" ", 1)[1]),) for text in line[:-1].split(";")])
    return out


def pieces(exe, mode, calls):
    """The pieces (x offset, y offset, m_total, ho, wo) of 1x1 convolutions: "pointwise", of the library's calls, "cut", cut at a given number of pixels."""
    return [[tuple(map(int, line.split()[i:i + 5])) for i in range(0, len(line.split()), 5)] for line in lines(exe, mode, calls)]
