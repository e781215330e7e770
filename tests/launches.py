"""Which kernels a call of the C ABI launches, asked on the CPU: `launches([call, ...])` runs the calls against
libtwn.so in a child process in which `launch_recorder.c` stands in for the HIP runtime.

A call is a dict: "fn" (gemm, conv, pair, bwd), "d" (fields of its descriptor, defaults below), and optionally
"env" (TWN_* overrides, re-read before the call), "env_late" (set without a re-read, after the workspace query),
"ws" (bytes of workspace; default: what the query says), "parts" (bwd: subset of "dx dw db"), "ptr" (name ->
address; distinct 1 TiB ranges by default), "residual" (True, or a pointer name).  The answer is {"rc", "need",
"launches": [{"kernel", "args", "grid", "block"}]}, `args` being the template arguments."""

import ctypes
import json
import os
import re
import struct
import subprocess
import sys
import tempfile

HERE = os.path.dirname(os.path.abspath(__file__))
LIB = os.path.join(os.path.dirname(HERE), "paper_1605_04711_amd", "libtwn.so")
F32, BF16 = 0, 1
CONV = ("N", "H", "W", "C", "O", "R", "S", "stride_h", "stride_w", "pad_h", "pad_w", "dil_h", "dil_w", "x_dtype", "y_dtype",
        "variant", "alpha_groups")
POINTERS = ("X", "W", "alpha", "Y", "ws", "dY", "dX", "dW", "db", "scale", "shift", "residual", "W1", "alpha1", "Y1", "residual1")


def conv(n, h, w, c, o, r, stride=1, pad=None, dil=1, groups=1, y=BF16, x=BF16, variant=None):
    pad = r // 2 if pad is None else pad
    return dict(N=n, H=h, W=w, C=c, O=o, R=r, S=r, stride_h=stride, stride_w=stride, pad_h=pad, pad_w=pad, dil_h=dil, dil_w=dil,
                x_dtype=x, y_dtype=y, variant=(3 if x == F32 else 0) if variant is None else variant, alpha_groups=groups)


def gemm(m, n, k, x=BF16, y=BF16, groups=1, ldx=0, ldy=0):
    return dict(M=m, N=n, K=k, x_dtype=x, y_dtype=y, variant=3 if x == F32 else 0, ldx=ldx, ldy=ldy, alpha_groups=groups)


def _pack(d):
    if "M" in d:
        return struct.pack("qiiiiixxxxqqixxxx", d["M"], d["N"], d["K"], d["x_dtype"], d["y_dtype"], d["variant"], d["ldx"], d["ldy"],
                           d["alpha_groups"])
    return struct.pack("17i", *[d[f] for f in CONV])


def launches(calls, lib=LIB):
    with tempfile.TemporaryDirectory() as tmp:
        so = os.path.join(tmp, "recorder.so")
        subprocess.check_call(["gcc", "-shared", "-fPIC", "-O1", "-o", so, os.path.join(HERE, "launch_recorder.c")])
        env = {k: v for k, v in os.environ.items() if not k.startswith("TWN_")}
        out = subprocess.run([sys.executable, os.path.abspath(__file__), so, lib], input=json.dumps(calls), text=True, check=True,
                             stdout=subprocess.PIPE, env=env).stdout
    answers = json.loads(out)
    found = [l for a in answers for l in a["launches"]]
    names = subprocess.run(["c++filt"], input="".join(l["name"] + "\n" for l in found), text=True, check=True,
                           stdout=subprocess.PIPE).stdout.splitlines()
    for l, name in zip(found, names):
        l["kernel"], args = re.search(r"(\w+_kernel)(<[^(]*>)?\(", name).groups()
        l["args"] = [] if args is None else [a.strip() for a in args[1:-1].split(",")]
    return answers


def _run(recorder, L, call):
    vp, i32, sz, f32 = ctypes.c_void_p, ctypes.c_int32, ctypes.c_size_t, ctypes.c_float
    env = call.get("env", {})
    os.environ.update({k: str(v) for k, v in env.items()})
    L.twn_reload_env()
    d = _pack(call["d"])
    d1 = _pack(call["d1"]) if "d1" in call else None
    p = {name: (i + 1) << 40 for i, name in enumerate(POINTERS)}
    p.update(call.get("ptr", {}))

    def query(name):
        fn = getattr(L, name)
        fn.restype, fn.argtypes = sz, [vp]
        return int(fn(d))

    need = {"gemm": lambda: query("twn_gemm_fwd_workspace_bytes"), "conv": lambda: query("twn_conv2d_fwd_workspace_bytes"),
            "bwd": lambda: query("twn_conv2d_bwd_ste_workspace_bytes"), "pair": lambda: 0}[call["fn"]]()
    os.environ.update({k: str(v) for k, v in call.get("env_late", {}).items()})
    ws = call.get("ws", need)

    def epilogue(key):
        r = call.get(key)
        return struct.pack("PPPi4x", 0, 0, p[key if r is True else r], 0) if r else None

    recorder.recorder_clear()
    if call["fn"] in ("gemm", "conv"):
        fn = getattr(L, "twn_gemm_fwd" if call["fn"] == "gemm" else "twn_conv2d_fwd")
        fn.restype, fn.argtypes = i32, [vp] * 7 + [sz, vp]
        rc = fn(d, p["X"], p["W"], p["alpha"], epilogue("residual"), p["Y"], p["ws"] if ws else None, ws, None)
    elif call["fn"] == "pair":
        fn = L.twn_conv2d_fwd_pair
        fn.restype, fn.argtypes = i32, [vp] * 12
        rc = fn(d, d1, p["X"], p["W"], p["alpha"], epilogue("residual"), p["Y"], p["W1"], p["alpha1"], epilogue("residual1"),
                p["Y1"], None)
    else:
        parts = call.get("parts", "dx dw db").split()
        fn = L.twn_conv2d_bwd_ste
        fn.restype, fn.argtypes = i32, [vp] * 8 + [f32, vp, sz, vp]
        rc = fn(d, p["X"], p["dY"], p["W"], p["alpha"], p["dX"] if "dx" in parts else None, p["dW"] if "dw" in parts else None,
                p["db"] if "db" in parts else None, 0.0, p["ws"] if ws else None, ws, None)
    got = []
    for i in range(recorder.recorder_count()):
        name = recorder.recorder_name(i).decode()
        dims = (ctypes.c_uint32 * 6)()
        recorder.recorder_grid(i, dims)
        got.append({"name": name, "grid": list(dims[:3]), "block": list(dims[3:])})
    for k in list(env) + list(call.get("env_late", {})):
        os.environ.pop(k, None)
    return {"rc": int(rc), "need": need, "launches": got}


def _main():
    recorder = ctypes.CDLL(sys.argv[1], mode=ctypes.RTLD_GLOBAL)
    recorder.recorder_name.restype = ctypes.c_char_p
    L = ctypes.CDLL(sys.argv[2])
    L.twn_reload_env.restype = None
    json.dump([_run(recorder, L, c) for c in json.load(sys.stdin)], sys.stdout)


if __name__ == "__main__":
    _main()
