"""The window pass and the split search run on the CPU, from the GPU library's
own sources, with the lanes of a workgroup as fibers (lanes.cpp)."""
from __future__ import annotations

import ctypes as C
import hashlib
import os
import subprocess

import numpy as np

from oracle import oracle as O

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(os.path.dirname(HERE))
CSRC = os.path.join(ROOT, "paper_2609_34244_amd", "csrc")
BUILD = os.path.join(HERE, "_build")
SOURCES = ["profile.cpp", "windows.hip", "search.hip", "evaluate.hip", "stage_cost.h", "heddle_internal.h", "device_common.h", "dp_common.h", "validate.h",
           "exact_math.h"]
LDS = 160 * 1024
SAMPLES, LEFT_HEAD = 64, 130         # kSamples, kLeftHead


class SplitRun(C.Structure):
    _fields_ = [("cus", C.c_int32), ("max_lds", C.c_int32), ("preset_on", C.c_int32), ("preset", C.c_uint32), ("need", C.c_float), ("need_slow", C.c_float), ("sweeps", C.c_int32), ("other", C.c_int32),
                ("placed", C.c_int32), ("lt", C.c_int32), ("lim", C.c_int32), ("per_cu", C.c_int32), ("n_broken", C.c_int32), ("broken", C.c_char * 256)]


def build():
    """compile lanes.cpp over copies of the sources, once per content"""
    text = {f: open(os.path.join(CSRC, f)).read().replace("extern __shared__", "extern") for f in SOURCES}
    text["heddle.h"] = open(os.path.join(ROOT, "include", "heddle.h")).read()
    for f in ("lanes.cpp", "hip/hip_runtime.h"):
        text[f] = open(os.path.join(HERE, f)).read()
    text["hip/hip_runtime_api.h"] = "#include <hip/hip_runtime.h>\n"
    text["heddle_internal.h"] = text["heddle_internal.h"].replace("../../include/heddle.h", "heddle.h")
    tag = hashlib.sha256("".join(f + text[f] for f in sorted(text)).encode()).hexdigest()[:16]
    out = os.path.join(BUILD, tag + ".so")
    if not os.path.exists(out):
        src = os.path.join(BUILD, tag)
        os.makedirs(os.path.join(src, "hip"), exist_ok=True)
        for f, t in text.items():
            with open(os.path.join(src, f), "w") as h:
                h.write(t)
        tmp = f"{out}.{os.getpid()}"
        subprocess.run(["g++", "-O2", "-g", "-std=c++17", "-fPIC", "-shared", "-w", "-Wl,-Bsymbolic", "-I", src, "-o", tmp,
                        os.path.join(src, "lanes.cpp")], check=True)
        os.replace(tmp, out)
    return out


_lib = None


def lib():
    global _lib
    if _lib is None:
        L = C.CDLL(build())
        P = C.c_void_p
        L.heddle_load_profile.argtypes = [P, P]
        L.heddle_free_profile.argtypes = [P]
        L.heddle_last_error.restype = C.c_char_p
        L.lanes_split.argtypes = [P, C.c_int64, C.c_int32, P, P, P, C.c_int32, C.c_uint32, P, P, P, P, P]
        L.lanes_evaluate.argtypes = [P, C.c_int64, C.c_int32, P, P, P, C.c_int32, C.c_uint32, P, P, P, P, P, P]
        L.lanes_left_template.argtypes = [P, C.c_int64, C.c_int64]
        L.lanes_left_template.restype = C.c_int64
        _lib = L
    return _lib


def split(w, flags=0, cus=1, max_lds=LDS, preset=None, other=0, need=0, need_slow=0, sweeps=0):
    """Window pass and split search over a workload. Returns the outputs that
    the search writes, `left` (the templates it left to the split kernel) and
    what it found broken (None: every stated condition held)."""
    L = lib()
    prof, h = O.OracleProfile(w.profile), C.c_void_p()         # the descriptor has the same layout
    assert L.heddle_load_profile(prof.ref, C.byref(h)) == 0, L.heddle_last_error()
    m = np.ascontiguousarray(w.m, np.int32)
    n, s_max = w.stages.shape
    t = np.float32 if flags & O.F_FP32 else np.int64
    bn, ly, st = np.empty((n, len(m)), t), np.empty((n, len(m), s_max), np.uint8), np.empty((n, len(m)), np.uint8)
    left = np.zeros(n + LEFT_HEAD, np.uint32)
    r = SplitRun(cus=cus, max_lds=max_lds, preset_on=preset is not None, preset=preset or 0, other=other, need=need, need_slow=need_slow, sweeps=sweeps)
    d = lambda a: a.ctypes.data
    ns, recs = np.ascontiguousarray(w.n_stages, np.uint8), np.ascontiguousarray(w.stages, np.uint32)
    rc = L.lanes_split(h, n, s_max, d(ns), d(recs), d(m), len(m), flags, d(bn), d(ly), d(st), d(left), C.addressof(r))
    err = L.heddle_last_error().decode(errors="replace") if rc else ""
    L.heddle_free_profile(h)
    return {"rc": rc, "error": err, "bottleneck": bn, "layers": ly, "status": st, "left_count": int(left[0]),
            "left": left[LEFT_HEAD:LEFT_HEAD + min(int(left[0]), n)], "ran": int(left[1]),
            "counted": int(left[2:2 + SAMPLES].sum()), "counted_stages": int(left[2 + SAMPLES:LEFT_HEAD].sum()), "broken": r.broken.decode() if r.n_broken else None,
            "n_broken": r.n_broken, "tables_in_lds": bool(r.lt), "limits_in_lds": bool(r.lim), "per_cu": r.per_cu}


def evaluate(w, flags, bottleneck, layers, status, max_lds=LDS):
    """Evaluate over given splits: (iter, peak memory, status, what broke or None)"""
    L = lib()
    prof, h = O.OracleProfile(w.profile), C.c_void_p()
    assert L.heddle_load_profile(prof.ref, C.byref(h)) == 0, L.heddle_last_error()
    m, ns, recs = (np.ascontiguousarray(x, t) for x, t in ((w.m, np.int32), (w.n_stages, np.uint8), (w.stages, np.uint32)))
    it, pk, st = np.empty_like(bottleneck), np.empty(bottleneck.shape, np.int64), np.array(status)
    r, d = SplitRun(cus=1, max_lds=max_lds), lambda a: a.ctypes.data
    rc = L.lanes_evaluate(h, w.n, recs.shape[1], d(ns), d(recs), d(m), len(m), flags, d(bottleneck), d(layers), d(st), d(it),
                          d(pk), C.addressof(r))
    L.heddle_free_profile(h)
    assert rc == 0
    return it, pk, st, r.broken.decode() if r.n_broken else None


def assert_split(w, g, flags, ctx=""):
    """the outputs of split() equal the oracle's wherever the search did not
    leave the template to the split kernel; returns how many it left"""
    o = O.price_plans(O.OracleProfile(w.profile), w.n_stages, w.stages, w.m, flags)
    assert g["rc"] == 0, g["error"]
    assert g["broken"] is None, f"{ctx}: {g['n_broken']} times, first {g['broken']}"
    own = np.ones(w.n, bool)
    own[g["left"]] = False
    st = o["status"]
    if flags & O.F_COMPUTE_ONLY:                               # fit is Evaluate's to check then
        st = np.where((st == 8) & (o["layers"].sum(-1) > 0), 0, st)
    for k, want in (("status", st), ("layers", o["layers"]), ("bottleneck", o["bottleneck"])):
        bad = np.argwhere((g[k] != want)[own])
        assert len(bad) == 0, f"{ctx}: {k} differs at {len(bad)} places, first {tuple(bad[0])}"
    return int((~own).sum())
