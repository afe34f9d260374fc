"""Runs the library's host path (validation, planning, workspaces, launch shapes) without a GPU.

``host_device.cpp`` stands in for the HIP runtime: device memory is host memory, launches are checked against the
launch limits, and nothing runs.  It has to be bound before the library, so every test body runs in a
child process: a test calls ``in_child(module, function, *args)`` and the child calls that function.
"""
import ctypes
import json
import os
import subprocess
import sys

import numpy as np

TESTS = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(TESTS)
_so = None


def build(tmp_path_factory) -> str:
    global _so
    if _so is None:
        out = str(tmp_path_factory.mktemp("host_device") / "libhost_device.so")
        subprocess.run(["g++", "-O1", "-std=c++17", "-shared", "-fPIC", os.path.join(TESTS, "host_device.cpp"), "-o", out],
                       check=True)
        _so = out
    return _so


def in_child(so: str, module: str, function: str, *args):
    code = (f"import sys; sys.path[:0] = [{ROOT!r}, {TESTS!r}]; import host_device as h; h.bind({so!r}); "
            f"import json, {module} as m; print('\\n@' + json.dumps(m.{function}(*json.loads({json.dumps(args)!r}))))")
    r = subprocess.run([sys.executable, "-c", code], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stderr[-4000:]
    return json.loads(r.stdout.rsplit("\n@", 1)[1])


# ---- in the child ----

_host = None


def bind(so: str) -> None:
    global _host
    _host = ctypes.CDLL(so, mode=ctypes.RTLD_GLOBAL)
    for f in ("host_live_bytes", "host_news", "host_launches"):
        getattr(_host, f).restype = ctypes.c_int64


def live_bytes() -> int:
    return _host.host_live_bytes()


def news() -> int:
    return _host.host_news()


class Layer:
    """A layer of zero codes and scales of one; ``conv`` is (cin, kernel, stride, pad, H, W)."""

    def __init__(self, C_out, K=0, M=2, B=8, g=8, max_n=1, x="f16", y="f16", cb="f16", tile="f16", conv=None):
        from paper_2506_05960_amd import aq
        self.aq = aq
        geom, per = None, 1
        if conv is not None:
            cin, k, stride, pad, H, W = conv
            geom = type("Conv", (), dict(cin=cin, kh=k, kw=k, stride=stride, pad=pad, H=H, W=W))
            K = cin * k * k
            per = ((H + 2 * pad - k) // stride + 1) * ((W + 2 * pad - k) // stride + 1)
        books = np.zeros((M, 1 << B, g), {"f16": np.float16, "f32": np.float32, "bf16": np.uint16}[cb])
        codes = np.zeros((C_out, K // g, M), np.uint8 if B <= 8 else np.uint16)
        desc = aq.make_desc(C_out, K, cb, x, y, tile, max_n * per, geom)
        self.handle = aq.aq_layer_create(desc, books, codes, np.ones(C_out, np.float32), g, M, B)
        self.x_scales = 4096 if x == "i8" else 0

    def set(self, **options):
        for k, v in options.items():
            self.aq.aq_layer_set_option(self.handle, self.aq.OPTION_CODES[k], v)
        return self

    def describe(self, n) -> dict:
        return self.aq.aq_layer_describe(self.handle, n)

    def forward(self, n, static=False):
        """Kernels of a forward (nothing reads the pointers), or the status it is refused with."""
        f = self.aq.aq_layer_forward_static if static else self.aq.aq_layer_forward
        try:
            f(self.handle, 4096, self.x_scales, 4096, n, 0)
        except self.aq.AQError as e:
            return self.aq.STATUS_NAMES[e.status]
        return [k.split("<")[0] for k in self.aq.aq_layer_last_launches(self.handle)[1]]

    def grad(self, n, dtype="f16"):
        """Kernels of a codebook gradient with their template arguments, or the status it is refused with."""
        try:
            self.aq.aq_layer_codebook_grad(self.handle, 4096, 4096, dtype, 4096, n, 0)
        except self.aq.AQError as e:
            return self.aq.STATUS_NAMES[e.status]
        return self.aq.aq_layer_last_launches(self.handle)[1]

    def close(self):
        self.aq.aq_layer_destroy(self.handle)


def launches(call):
    """Result of ``call()``, and grid, block and dynamic LDS bytes of each kernel it launched."""
    _host.host_reset_launches()
    result, out = call(), []
    for i in range(_host.host_launches()):
        one = (ctypes.c_uint64 * 7)()
        _host.host_launch(ctypes.c_int64(i), one)
        out.append(list(one))
    return result, out
