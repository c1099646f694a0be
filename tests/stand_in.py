"""The library's host code on a counting stand-in for the HIP runtime
(hip_stand_in.c): run(body) executes `body` in a fresh interpreter in which
libnavsim.so's runtime calls are the stand-in's.  In the body: lib (the
library), ns (the binding), np, C, a Counts() of the calls since clear(),
launches() by kernel name, and helpers to make handles."""
import os
import subprocess
import sys
import textwrap

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)

PRELUDE = r'''
import ctypes as C, sys, types
sys.modules["torch"] = types.ModuleType("torch")  # the binding's imports only name it
R = C.CDLL(sys.argv[1], mode=C.RTLD_GLOBAL)
R.stand_in_launch.restype = C.c_char_p
import numpy as np
from collections import namedtuple
from paper_2606_15846_amd import navsim as ns
from paper_2606_15846_amd import reset_proposal as rpm
from workloads import configs, maps as gm
lib = rpm._lib()
Counts = namedtuple("Counts", "launches malloc free sync copy")

def clear():
    R.stand_in_clear()

def counts():
    v = (C.c_int * 5)()
    R.stand_in_counts(v)
    return Counts(*v)

def names(raw):
    import re, subprocess
    out = subprocess.run(["c++filt"], input="\n".join(raw), capture_output=True, text=True).stdout
    return [re.search(r"(\w+_kernel(?:<[^(]*>)?)\(", n).group(1) for n in out.split("\n") if n]

def launches():
    """Kernel names (without namespace, with template arguments) since clear()."""
    return names([R.stand_in_launch(i).decode() for i in range(counts().launches)])

def kernels():
    """Names of the kernels in the library."""
    R.stand_in_kernel.restype = C.c_char_p
    raw = []
    while R.stand_in_kernel(len(raw)):
        raw.append(R.stand_in_kernel(len(raw)).decode())
    return names(raw)

def handle(n, sides, beams=36, sectors=36, res=0.05, rmax=3.5, **k):
    """A handle with one map per (W, H) of `sides`, loaded and reset."""
    d = dict(num_envs=n, num_beams=beams, num_sectors=sectors, fov_rad=6.2831853, max_range_m=rmax,
             dt_s=0.1, footprint=0, radius_m=0.18, v_min=0.0, v_max=0.5, w_min=-1.0, w_max=1.0)
    d.update(k)
    h = ns.navsim_create(configs.make_config(**d))
    load(h, n, sides, res)
    obs = np.zeros((n, sectors + 4), np.float32)
    assert lib.navsim_reset(h, None, obs.ctypes.data, None) == 0
    return h

def load(h, n, sides, res=0.05):
    occ = [np.pad(np.zeros((b - 2, a - 2), np.uint8), 1, constant_values=1) for a, b in sides]
    ns.navsim_load_maps(h, occ, [res] * len(occ), configs.contiguous_env_map(n, len(occ)))

def step(h, n, sectors=36, final=True):
    f = lambda *s: np.zeros(s, np.float32)
    u = np.zeros(n, np.uint8)
    o, fo = f(n, sectors + 4), f(n, sectors + 4)
    return lib.navsim_step(h, f(n, 2).ctypes.data, o.ctypes.data, f(n).ctypes.data, u.ctypes.data,
                           u.ctypes.data, fo.ctypes.data if final else None, None)

def proposer(h, **k):
    c = dict(rpm.DEFAULT, **k)
    rc = rpm.RPConfig(**{q: c[q] for q, _ in rpm.RPConfig._fields_})
    r = C.c_void_p()
    ns._check(lib.navsim_rp_create(h, C.byref(rc), C.byref(r)))
    return r

def propose(r, n, proposals, tries, noalloc=False):
    i = [np.zeros(max(n, 1), np.int32) for _ in range(7)]
    pose = np.zeros((max(n, 1), 5), np.float32)
    fn = lib.navsim_rp_propose_noalloc if noalloc else lib.navsim_rp_propose
    return fn(r, n, *[a.ctypes.data for a in i[:4]], proposals, tries, pose.ctypes.data,
              *[a.ctypes.data for a in i[4:]], None, None)
'''

_SO = None


def _stand_in(tmp):
    global _SO
    if _SO is None:
        _SO = os.path.join(str(tmp), "hip_stand_in.so")
        subprocess.run(["gcc", "-O1", "-std=c11", "-shared", "-fPIC", "-w",
                        os.path.join(HERE, "hip_stand_in.c"), "-o", _SO], check=True)
    return _SO


def run(tmp, body):
    code = PRELUDE + textwrap.dedent(body) + '\nprint("done")\n'
    r = subprocess.run([sys.executable, "-c", code, _stand_in(tmp)], cwd=ROOT, text=True,
                       capture_output=True, timeout=300, env=dict(os.environ, PYTHONPATH=ROOT))
    assert r.returncode == 0 and r.stdout.rstrip().endswith("done"), \
        f"exit {r.returncode}\n{r.stdout}\n{r.stderr}"
    return r.stdout
