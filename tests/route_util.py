"""Which kernels a call launches, asked of the library's host side without a GPU (tests/route_driver.c)."""
import collections
import os
import re
import subprocess

from conftest import ROOT

PROB, LOGIT, BF16 = 0, 1, 2
Route = collections.namedtuple("Route", "status workspace launches")   # launches: [(kernel, grid, threads)]
Launch = collections.namedtuple("Launch", "kernel grid threads")


def build_driver(path):
    from paper_2506_03206_amd import build, rdk
    if not os.path.exists(rdk.LIB_PATH):
        build.build()
    exe = str(path / "route_driver")
    made = subprocess.run(["gcc", "-std=c99", "-Wall", "-O1", "-rdynamic", "-I", os.path.join(ROOT, "include"),
                           os.path.join(ROOT, "tests", "route_driver.c"), rdk.LIB_PATH, "-Wl,-rpath," + os.path.dirname(rdk.LIB_PATH),
                           "-Wl,--allow-shlib-undefined", "-o", exe], capture_output=True, text=True)
    assert made.returncode == 0, made.stderr
    return exe


def plain(name):
    """The kernel's own name and its template arguments, out of a mangled one: exact_bf16_kernel<4,1,0>."""
    found = re.match(r"_ZN3rdk12_GLOBAL__N_1(\d+)(.*)", name) or re.match(r"_ZN3rdk(\d+)(.*)", name)
    own, rest = found.group(2)[:int(found.group(1))], found.group(2)[int(found.group(1)):]
    args = re.match(r"I((?:L[ib]n?\d+E|LN\w*?E\d+E)*)", rest)
    values = re.findall(r"(n?\d+)E(?=L|$)", args.group(1)) if args else []
    values = [v.replace("n", "-") for v in values]
    return own + ("<%s>" % ",".join(values) if values else "")


def routes(exe, lines):
    run = subprocess.run([exe], input="\n".join(lines) + "\n", capture_output=True, text=True, timeout=300)
    assert run.returncode == 0, run.stdout[-2000:] + run.stderr
    out = []
    for text in run.stdout.splitlines():
        first, *mid, status = text.split(";")
        launches = [Launch(plain(m.split()[0]), tuple(map(int, m.split()[1:4])), int(m.split()[4])) for m in mid]
        out.append(Route(int(status), int(first.split()[1]), launches))
    assert len(out) == len(lines)
    return out
