"""TEST INFRASTRUCTURE ONLY: the replay kernels compiled for the host (64 lanes as cooperative
fibers, guard bands around every buffer) and a ctypes loader for that build.  Used by the CPU
tests to check the kernels' indexing and decisions without a GPU; never by the product."""
import ctypes
import os
import subprocess

import numpy as np

_HERE = os.path.dirname(os.path.abspath(__file__))
_SRC = os.path.join(_HERE, "emu_replay.cpp")
_LIB = os.path.join(_HERE, "libemu.so")
_CSRC = os.path.join(_HERE, "..", "..", "paper_2401_08156_amd", "csrc")
_DEPS = [_SRC, os.path.join(_HERE, "wave_hw_emu.hpp")] + [
    os.path.join(_CSRC, f) for f in ("wave_ops.hpp", "replay_plan.hpp", "replay_kernels.hpp", "replay_fine.hpp", "selftest.hpp")]


def build(force=False):
    if not force and os.path.exists(_LIB) and all(os.path.getmtime(_LIB) >= os.path.getmtime(d) for d in _DEPS):
        return _LIB
    subprocess.run(["g++", "-O1", "-g", "-std=c++17", "-shared", "-fPIC", "-Wall", "-Wno-unused", "-Wno-unknown-pragmas", "-Wno-restrict",
                    "-o", _LIB, _SRC], check=True)
    return _LIB


_lib = None


def lib():
    global _lib
    if _lib is None:
        _lib = ctypes.CDLL(build())
        vp = ctypes.c_void_p
        _lib.emu_replay.restype = ctypes.c_int
        _lib.emu_replay.argtypes = [vp, vp, vp, vp, vp, vp]
        _lib.emu_selftest.restype = ctypes.c_uint
        _lib.emu_plan.restype = ctypes.c_int
        _lib.emu_plan.argtypes = [vp, ctypes.c_int, vp]
    return _lib


class Plan(ctypes.Structure):
    """What tests ask of a plan; slots: SLOTS_IN_LDS, SLOTS_IN_REGS or SLOTS_IN_MEM."""
    _fields_ = [("fine", ctypes.c_uint32), ("slots", ctypes.c_uint32), ("tbl_ws", ctypes.c_uint32), ("has_retry", ctypes.c_uint32),
                ("lds_bytes", ctypes.c_uint32 * 2), ("mem_stride", ctypes.c_uint64 * 2), ("cost", ctypes.c_uint64)]


SLOTS_IN_LDS, SLOTS_IN_REGS, SLOTS_IN_MEM = 0, 1, 2


def plan(cfg, in_lds=False, tables_in_mem=-1):
    """(VMS_OK or an error code, the plan the library makes for cfg; in_lds: where there is no memory for its tables).
    tables_in_mem: the one plan of the variant and table place that cfg names, with its slot tables (1) and its table of
    multi-chunk pBlocks (2) in global memory."""
    out = Plan()
    lib().emu_use_plan(PLAN_IN_LDS if in_lds else PLAN_OF_LIBRARY)
    return lib().emu_plan(ctypes.byref(cfg), tables_in_mem, ctypes.byref(out)), out


PLAN_OF_LIBRARY, PLAN_POOL_IN_MEM, PLAN_SMALL, PLAN_IN_LDS = 0, 1, 2, 3


def replay(events, cfg, stats_dtype, n_events=None, pool_in_mem=False, small=False, in_lds=False):
    """events: uint64[n_traces, max_events]; cfg: the binding's vms_config; pool_in_mem: the plan of a large batch with
    all tables in the workspace (cfg names VMS_TABLES_WORKSPACE_ALL); small: the plan that needs least workspace;
    in_lds: the one without tables in global memory.
    Returns (dec_split, dec_vms, stats[2, n_traces])."""
    ev = np.ascontiguousarray(events, dtype=np.uint64)
    assert ev.shape == (cfg.n_traces, cfg.max_events)
    ds, dv = np.zeros_like(ev), np.zeros_like(ev)
    st = np.zeros((2, cfg.n_traces), dtype=stats_dtype)
    ne = None if n_events is None else np.ascontiguousarray(n_events, dtype=np.uint32)
    lib().emu_use_plan(PLAN_POOL_IN_MEM if pool_in_mem else PLAN_SMALL if small else PLAN_IN_LDS if in_lds else PLAN_OF_LIBRARY)
    rc = lib().emu_replay(ctypes.byref(cfg), ev.ctypes.data, None if ne is None else ne.ctypes.data,
                          ds.ctypes.data, dv.ctypes.data, st.ctypes.data)
    if rc != 0:
        raise RuntimeError("emu_replay: %d" % rc)
    return ds, dv, st
