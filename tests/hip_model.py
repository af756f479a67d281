"""Runs the library's host code against a model of the HIP runtime (hip_model.cpp), in a process of its own without a GPU.
A test marked @in_model receives the Model; its body runs in a child process that loads the model in the runtime's place."""
from __future__ import annotations

import ctypes as C
import functools
import os
import subprocess
import sys

import numpy as np

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
SOURCE = os.path.join(HERE, "hip_model.cpp")
LIB = os.path.join(HERE, "_build", "hip_model.so")
PER_THREAD = 2          # hipStreamPerThread


def build():
    deps = [SOURCE, os.path.join(ROOT, "paper_2403_19708_amd", "csrc", "ca_internal.h")]
    if not os.path.exists(LIB) or os.path.getmtime(LIB) < max(os.path.getmtime(d) for d in deps):
        os.makedirs(os.path.dirname(LIB), exist_ok=True)
        mine = f"{LIB}.{os.getpid()}"
        subprocess.run(["g++", "-O1", "-std=c++17", "-fPIC", "-shared", "-w", "-I/opt/rocm/include", SOURCE, "-Wl,-soname,libamdhip64.so.7", "-o", mine],
                       check=True)
        os.replace(mine, LIB)


def in_model(test):
    @functools.wraps(test)
    def run_in_child(**params):
        build()
        code = f"import sys; sys.path[:0] = [{ROOT!r}, {HERE!r}]; import hip_model; hip_model.child({test.__module__!r}, {test.__name__!r}, {params!r})"
        done = subprocess.run([sys.executable, "-c", code], capture_output=True, text=True, timeout=120)
        assert done.returncode == 0, done.stdout + done.stderr
    run_in_child.in_model = test
    del run_in_child.__wrapped__
    import inspect
    run_in_child.__signature__ = inspect.Signature([p for p in inspect.signature(test).parameters.values()][1:])
    return run_in_child


def child(module, name, params):
    model = Model()                     # before the library, which then finds the runtime it needs already loaded
    getattr(__import__(module), name).in_model(model, **params)


class Model:
    def __init__(self):
        self.lib = C.CDLL(LIB, mode=C.RTLD_GLOBAL)
        for f, res, args in (("model_alloc", C.c_void_p, [C.c_size_t, C.c_int]), ("model_what", C.c_char_p, [C.c_int]),
                             ("model_stream", C.c_void_p, [C.c_int]), ("model_stream_behind", C.c_int, [C.c_void_p, C.c_int]),
                             ("model_capture", C.c_int, [C.c_void_p, C.c_int]), ("model_device_bytes", C.c_size_t, []),
                             ("model_attn_pointer", C.c_void_p, [C.c_int, C.c_int]),
                             ("model_move_pointer", C.c_void_p, [C.c_int, C.c_int, C.c_int])):
            getattr(self.lib, f).restype, getattr(self.lib, f).argtypes = res, args

    def device(self, d):
        assert self.lib.hipSetDevice(d) == 0

    def current(self):
        d = C.c_int()
        assert self.lib.hipGetDevice(C.byref(d)) == 0
        return d.value

    def stream(self):
        s = C.c_void_p()
        assert self.lib.hipStreamCreateWithFlags(C.byref(s), 1) == 0
        return s.value

    def alloc(self, size, kind=0):
        return self.lib.model_alloc(size, kind)

    def queued(self, call):
        """the operations queued while call() runs"""
        before = self.lib.model_ops()
        call()
        return list(range(before, self.lib.model_ops()))

    def what(self, op):
        return self.lib.model_what(op).decode()

    def named(self, ops, text):
        return [op for op in ops if text in self.what(op)]

    def done(self, op):
        return bool(self.lib.model_done(op))

    def behind(self, op, other):
        return bool(self.lib.model_behind(op, other))

    def stream_behind(self, stream, op):
        return bool(self.lib.model_stream_behind(stream, op))


class Turn:
    """A context and the memory of one batch: hist / new tokens per conversation, tier kind as model_alloc's."""

    def __init__(self, m, hist, new, tier=0, device=0, layers=1, heads=(4, 2, 128), tier_rows=None, **cfg):
        import paper_2403_19708_amd as ca
        self.m, self.hist, self.new = m, np.array(hist, np.int32), np.array(new, np.int32)
        hq, hkv, d = heads
        n = len(hist)
        m.device(device)
        pages = (self.hist + self.new + 15) // 16
        self.num_pages = int(pages.sum()) + 1
        self.table = np.full((n, int(pages.max())), -1, np.int32)
        at = 0
        for c in range(n):
            self.table[c, :pages[c]] = range(at, at + pages[c])
            at += pages[c]
        self.row = hkv * d * 2
        pool = self.num_pages * 16 * self.row
        self.kp, self.vp = m.alloc(pool), m.alloc(pool)
        rows = self.hist + self.new if tier_rows is None else np.array(tier_rows)
        self.tk, self.tv = ([m.alloc(int(r) * self.row, tier) for r in rows] for _ in range(2))
        total = int(self.new.sum())
        self.q, self.out = m.alloc(total * hq * d * 2), m.alloc(total * hq * d * 2)
        self.nk, self.nv = m.alloc(total * self.row), m.alloc(total * self.row)
        self.scale = d ** -0.5
        self.ctx = ca.Context(ca.Config(n_layers=layers, n_q_heads=hq, n_kv_heads=hkv, head_dim=d, max_positions=65536, max_seqs=n,
                                        max_batch_kv_tokens=int((self.hist + self.new).sum()) + 64, max_batch_q_tokens=total + 16, device=device, **cfg))

    def rebase(self, stream=None, **kw):
        self.ctx.rope_rebase(self.hist, np.zeros_like(self.hist), self.new, self.table, self.num_pages, stream, **kw)

    def load(self, layer=0):
        self.ctx.kv_load_layer(layer, self.tk, self.tv, self.kp, self.vp)

    def append(self, stream=None, layer=0):
        self.ctx.kv_append_layer(layer, self.nk, self.nv, self.kp, self.vp, stream)

    def attn(self, stream=None, layer=0, static=False):
        call = self.ctx.cached_prefill_attn_static if static else self.ctx.cached_prefill_attn
        call(layer, self.q, self.kp, self.vp, self.out, self.scale, stream)

    def save(self, stream=None, layer=0, **kw):
        self.ctx.kv_save_layer(layer, self.kp, self.vp, self.tk, self.tv, after_stream=stream, **kw)

    def append_save(self, stream=None, layer=0):
        self.ctx.kv_append_save_layer(layer, self.nk, self.nv, self.kp, self.vp, self.tk, self.tv, stream)
