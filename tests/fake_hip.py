"""The library's host side on the CPU, over a HIP runtime that only writes launches down (tests/san/fake_hip.cpp).

Run as a script in a process of its own (the runtime has to come before everything else that uses HIP, so nothing here imports
torch): `python fake_hip.py FAKE LIB`, with a JSON list of steps on stdin, and a JSON list of results on stdout.  Steps:

  {"do": "ctx", "bytes": n}                        a new context with a workspace of n bytes (0: clada_workspace_bytes of "sizes")
  {"do": "option", "name": .., "value": ..}
  {"do": "stack" | "decode", "d", "F", "L", "B", "kind", "dtype", "dense"}
  {"do": "prefix", "d", "F", "T", "kind"} / {"do": "calibrate", "n": ..} / {"do": "search", "d", "F", "T", "bound", "n_probes"}
  {"do": "fail", "in": n} / {"do": "capturing", "on": 0 | 1}

A result is {"status": .., "launches": [[kernel, gx, gy, gz, bx, on a lane's stream], ..], "created": streams and events}."""
import ctypes as C
import json
import os
import subprocess
import sys

KINDS = {"swiglu": 0, "relu": 1, "geglu": 2}
DTYPES = {"f32": 0, "bf16": 1}


class CLayer(C.Structure):
    _fields_ = [("w_gate", C.c_void_p), ("w_up", C.c_void_p), ("w_down", C.c_void_p), ("d", C.c_int32), ("d_ff", C.c_int32),
                ("dtype", C.c_int32), ("kind", C.c_int32), ("b_in", C.c_void_p), ("b_out", C.c_void_p)]


def build_runtime(folder):
    """Compiles the stand-in runtime; returns its path."""
    fake = os.path.join(str(folder), "libfake_hip.so")
    src = os.path.join(os.path.dirname(os.path.abspath(__file__)), "san", "fake_hip.cpp")
    subprocess.run(["g++", "-std=c++17", "-O1", "-shared", "-fPIC", "-I/opt/rocm/include", src, "-o", fake], check=True,
                   capture_output=True, text=True)
    return fake


def run_steps(fake, steps):
    """The steps in a child process over the runtime at the path `fake`."""
    here = os.path.dirname(os.path.abspath(__file__))
    import paper_2502_19078_amd as pkg
    if not os.path.exists(pkg.lib_path()):
        from paper_2502_19078_amd import build
        build.build()
    r = subprocess.run([sys.executable, os.path.join(here, "fake_hip.py"), fake, pkg.lib_path()], input=json.dumps(steps),
                       capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stderr[-2000:]
    return json.loads(r.stdout)


def _main(fake_path, lib_path):
    fake = C.CDLL(fake_path, mode=C.RTLD_GLOBAL)
    lib = C.CDLL(lib_path)
    fake.fake_take_log.restype = C.c_char_p
    lib.clada_workspace_bytes.restype = C.c_size_t
    vp = C.c_void_p
    buf = C.create_string_buffer(1 << 16)
    p = vp((C.addressof(buf) + 255) // 256 * 256)            # stands for every device pointer; nothing reads it
    ctx = vp()
    out = []
    for s in json.load(sys.stdin):
        do, st = s["do"], 0
        layer = None
        if "d" in s:
            layer = CLayer(p, p, p, s["d"], s["F"], DTYPES[s.get("dtype", "bf16")], KINDS[s.get("kind", "swiglu")], p, p)
        if do == "ctx":
            if ctx:
                lib.clada_destroy(ctx)
            n = s.get("bytes") or lib.clada_workspace_bytes(*[C.c_int32(v) for v in s["sizes"]])
            ctx = vp()
            st = lib.clada_create(C.byref(ctx), 0, C.c_size_t(n))
        elif do == "option":
            st = lib.clada_set_option(ctx, s["name"].encode(), C.c_int32(s["value"]))
        elif do == "stack":
            arr = (CLayer * s["L"])(*[layer] * s["L"])
            st = (lib.clada_dense_ffn_stack_decode(ctx, arr, s["L"], p, s["B"], p, None) if s.get("dense")
                  else lib.clada_sparse_ffn_stack_decode(ctx, arr, s["L"], p, s["B"], p, p, None, None))
        elif do == "decode":
            st = lib.clada_sparse_ffn_decode(ctx, C.byref(layer), p, s["B"], p, p, None, None, None, None)
        elif do == "prefix":
            outs = (C.c_void_p * 6)(*[p] * 6)
            st = lib.clada_prefix_stats(ctx, C.byref(layer), p, s["T"], p, outs, None)
        elif do == "calibrate":
            st = lib.clada_threshold_calibrate(ctx, p, C.c_int64(s["n"]), C.c_float(0.45), p, None)
        elif do == "search":
            st = lib.clada_threshold_search_cett(ctx, C.byref(layer), p, s["T"], C.c_float(s.get("bound", 0.2)), s.get("n_probes", 31), p, p, None)
        elif do == "fail":
            fake.fake_fail_launch(C.c_long(s["in"]))
        elif do == "capturing":
            fake.fake_capturing(s["on"])
        else:
            raise ValueError(do)
        rows = [r.split() for r in fake.fake_take_log().decode().splitlines()]
        out.append({"status": st, "launches": [[r[0]] + [int(v) for v in r[1:]] for r in rows],
                    "created": fake.fake_take_streams() + fake.fake_take_events()})
    json.dump(out, sys.stdout)


if __name__ == "__main__":
    _main(*sys.argv[1:3])
