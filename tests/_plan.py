"""Launch plans of the built library, without a device (tests/plan_driver)."""
import collections
import os
import subprocess

from paper_2206_11524_amd import lbm

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
ROCM = os.environ.get("ROCM_PATH", "/opt/rocm")
KNOBS = ("LBM_BOX", "LBM_TILE_X", "LBM_TILE_Y", "LBM_ZCHUNK", "LBM_BATCH_TILE_X", "LBM_BATCH_TILE_Y")
FORCING = {"shan-chen": 0, "guo": 1}

Plan = collections.namedtuple("Plan", "box tile zchunk nt group server cells")


def build_driver(name, out):
    """Compile tests/plan_driver/<name>.cpp against the library's own headers
    and link it to the built library."""
    pkg = os.path.dirname(lbm.LIB_PATH)
    cmd = ["g++", "-std=c++17", "-O1", "-Wall", "-Wextra", "-D__HIP_PLATFORM_AMD__", "-isystem",
           os.path.join(ROCM, "include"), "-I", os.path.join(ROOT, "include"), "-I", os.path.join(pkg, "csrc"),
           os.path.join(ROOT, "tests", "plan_driver", name + ".cpp"), "-rdynamic", "-L", pkg, "-lhmcsc",
           f"-Wl,-rpath,{pkg}", "-L", os.path.join(ROCM, "lib"), "-lamdhip64",
           f"-Wl,-rpath,{os.path.join(ROCM, 'lib')}", "-o", str(out)]
    r = subprocess.run(cmd, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    return str(out)


def run_driver(exe, args=(), text=None, env=None):
    e = {k: v for k, v in os.environ.items() if k not in KNOBS}
    e.update({k: str(v) for k, v in (env or {}).items()})
    r = subprocess.run([exe, *[str(a) for a in args]], input=text, capture_output=True, text=True, env=e, timeout=60)
    assert r.returncode == 0, (r.returncode, r.stderr)
    return r.stdout.splitlines()


def plans(exe, domains, env=None):
    """Plan of each (shape, storage, ncomp, c_ns, forcing)."""
    text = "".join("%d %d %d %d %d %d %d\n" % (*s, lbm.STORAGE[st], nc, cn, FORCING[fo])
                   for s, st, nc, cn, fo in domains)
    out = [tuple(map(int, line.split())) for line in run_driver(exe, text=text, env=env)]
    assert len(out) == len(domains)
    return [Plan(v[0:3] if v[0] else None, v[3:5], v[5], bool(v[6]), v[7:9], v[9:11], v[11]) for v in out]
