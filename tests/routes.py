"""Which kernels the library's calls launch, found without a GPU: a process of its own loads
launch_recorder.cpp in the place of the HIP runtime, makes the calls with addresses that nothing follows,
and reports the launches.

    routes([dict(fn="backward", n_in=16, n_out=16, grid=8, batch=256, grad_x=1, grad_coef=1), ...])

gives for every call (status, [(kernel, grid, threads, LDS bytes), ...]).  A call is a dict of
  fn         "forward", "forward_static", "backward", "hessian" or "workspace" (whose status is the size)
  n_in, n_out, grid, batch; dtype (0, 1, 2), layout (0, 1), flags (default 0)
  conv       (n, h, w, c_in, kh, kw, stride) instead of batch
  grad_x, grad_coef   which gradients a backward call is asked for (1 or 0)
  x, coef, y, gy, gx, gp   offsets in bytes added to the 256-byte aligned address of that buffer
  ws         the workspace's size (default: what the library asks for)
  pass_      which size "workspace" asks for
"""
import ctypes as C
import json
import os
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
LIBRARY = os.path.join(os.path.dirname(HERE), "paper_2509_07103_amd", "liblmkan.so")
_recorder = None


def recorder(folder):
    """The recorder, compiled into `folder`."""
    out = os.path.join(str(folder), "launch_recorder.so")
    subprocess.run(["g++", "-O1", "-std=c++17", "-shared", "-fPIC", "-o", out,
                    os.path.join(HERE, "launch_recorder.cpp")], check=True)
    return out


def routes(calls, recorder_path, library=LIBRARY):
    got = subprocess.run([sys.executable, os.path.abspath(__file__), recorder_path, library], input=json.dumps(calls),
                         capture_output=True, text=True)
    assert got.returncode == 0, got.stderr
    return [(status, [tuple(launch) for launch in launches]) for status, launches in json.loads(got.stdout)]


def names(launches):
    """Kernel names without their template arguments."""
    return [launch[0].split("<")[0] for launch in launches]


def variants(launches, kernel):
    """The template arguments with which `kernel` is launched, "" where it is no template."""
    return [launch[0][len(kernel):].strip("<>") for launch in launches if launch[0].split("<")[0] == kernel]


class _Desc(C.Structure):
    _fields_ = [(f, C.c_int32) for f in ("n_in", "n_out", "grid", "order", "dtype", "layout", "flags")]


class _Conv(C.Structure):
    _fields_ = [(f, C.c_int32) for f in ("n", "h", "w", "c_in", "kh", "kw", "stride")]


def _main():
    rec = C.CDLL(sys.argv[1], mode=C.RTLD_GLOBAL)
    lib = C.CDLL(sys.argv[2])
    rec.recorder_text.restype = C.c_char_p
    lib.lmkan_workspace_bytes.restype = C.c_size_t
    lib.lmkan_conv2d_rows.restype = C.c_int64
    at = {name: (i + 1) << 40 for i, name in enumerate(("x", "coef", "y", "gy", "gx", "gp", "ws"))}
    out = []
    for c in json.load(sys.stdin):
        d = _Desc(c["n_in"], c["n_out"], c["grid"], 2, c.get("dtype", 0), c.get("layout", 0), c.get("flags", 0))
        dp = C.byref(d)
        conv = _Conv(*c["conv"]) if c.get("conv") else None
        rows = lib.lmkan_conv2d_rows(C.byref(conv), None, None) if conv else c["batch"]
        geometry = C.byref(conv) if conv else C.c_int64(rows)
        fn = c["fn"]
        grad_x, grad_coef = c.get("grad_x", 1), c.get("grad_coef", 1)
        which = 0 if fn.startswith("forward") else 1 if grad_x and grad_coef else 2 if grad_x else 3
        need = lib.lmkan_workspace_bytes(dp, C.c_int64(rows), c.get("pass_", which))
        size = c.get("ws", need)
        p = {name: C.c_void_p(at[name] + c.get(name, 0) if name != "ws" else at["ws"]) for name in at}
        ws = p["ws"] if size else None
        rec.recorder_clear()
        if fn == "workspace":
            status = need
        elif fn == "forward":
            call = lib.lmkan_conv2d_forward if conv else lib.lmkan_forward
            status = call(dp, geometry, p["x"], p["coef"], p["y"], ws, C.c_size_t(size), None)
        elif fn == "forward_static":
            status = lib.lmkan_forward_static(dp, C.c_int64(rows), p["x"], p["coef"], p["y"], None)
        elif fn == "hessian":
            status = lib.lmkan_hessian_reg(dp, p["coef"], C.c_float(1.0), p["ws"], p["gp"] if grad_coef else None, None)
        else:
            call = lib.lmkan_conv2d_backward if conv else lib.lmkan_backward
            status = call(dp, geometry, p["x"], p["coef"], p["gy"], p["gx"] if grad_x else None,
                          p["gp"] if grad_coef else None, ws, C.c_size_t(size), None)
        launches = []
        for line in rec.recorder_text().decode().splitlines():
            name, grid, threads, lds = line.split("\t")
            launches.append((name, [int(v) for v in grid.split(",")], int(threads), int(lds)))
        out.append((status, launches))
    json.dump(out, sys.stdout)


if __name__ == "__main__":
    _main()
