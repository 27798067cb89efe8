"""Runs calls of the C ABI against the stand-in HIP runtime (_fake_hip.c) in a process of its own and reports their kernel
launches: `python -m tests._fake_hip stand_in.so < calls.json`.  A call is {"entry", "cfg": [moe_config fields], "T", and what
the entry takes besides}; "fail": index of the launch that fails.  Not collected by pytest."""
import ctypes as C
import json
import os
import re
import subprocess
import sys
import types

HERE = os.path.dirname(os.path.abspath(__file__))


class _Dim3(C.Structure):
    _fields_ = [("x", C.c_uint), ("y", C.c_uint), ("z", C.c_uint)]


def trace(calls, tmp_path):
    """[{status, launches: [{name, grid, block, args...}]}] of the calls, from a fresh process."""
    so = os.path.join(str(tmp_path), "fake_hip.so")
    if not os.path.exists(so):
        subprocess.run(["gcc", "-O1", "-shared", "-fPIC", os.path.join(HERE, "_fake_hip.c"), "-o", so], check=True)
    r = subprocess.run([sys.executable, "-m", "tests._fake_hip", so], input=json.dumps(calls), capture_output=True, text=True,
                       cwd=os.path.dirname(HERE), timeout=120)
    assert r.returncode == 0, r.stderr
    return json.loads(r.stdout)


def _int_at(arg, offset):
    return C.cast(arg + offset, C.POINTER(C.c_int32))[0]


def _details(name, args):
    """What the tests look at among a kernel's arguments."""
    if "gate_logits" in name:                       # GateArgs: three pointers, T d m m_pad K score_fn, four pointers, n_slice
        return {"T": _int_at(args[0], 24), "n_slice": _int_at(args[0], 80)}
    if "combine" in name:
        return {"T": _int_at(args[5], 0), "planes": _int_at(args[10], 0)}
    return {}


def _main():
    stub = types.ModuleType("torch")
    stub.Tensor = object
    sys.modules["torch"] = stub                     # torch brings the real HIP runtime into the process
    fake = C.CDLL(sys.argv[1], mode=C.RTLD_GLOBAL)
    import importlib.util
    spec = importlib.util.spec_from_file_location("binding", os.path.join(HERE, "..", "paper_2507_17133_amd", "binding.py"))
    B = importlib.util.module_from_spec(spec)
    sys.modules["binding"] = B
    spec.loader.exec_module(B)
    L = B.lib()
    launches, fail = [], [-1]

    def on_launch(name, grid, block, lds, args):
        name = name.decode()
        # _ZN4bmoe<length><name>...: the length tells the name from what follows it
        m = re.match(r"_ZN4bmoe(\d+)", name)
        plain = name[m.end():m.end() + int(m.group(1))] if m else name
        launches.append(dict({"name": plain, "symbol": name, "grid": grid.x * grid.y * grid.z, "block": block.x, "lds": lds},
                             **_details(plain, args)))
        return 1 if len(launches) - 1 == fail[0] else 0

    cb = C.CFUNCTYPE(C.c_int, C.c_char_p, _Dim3, _Dim3, C.c_size_t, C.POINTER(C.c_void_p))(on_launch)
    fake.fake_on_launch(cb)
    mem = [0x100000 * i for i in range(1, 40)]      # never read or written
    p = lambda i: C.c_void_p(mem[i])
    w = lambda i: C.byref(B.moe_ffn_weights(mem[i], mem[i + 1], mem[i + 2]))
    out = []
    for c in json.load(sys.stdin):
        cfg = B.moe_config(*c["cfg"])
        b = C.byref(cfg)
        T, thr, full = c["T"], C.c_double(c.get("threshold", 1.0)), c.get("full", 0)
        shared = w(16) if cfg.n_shared else None
        route = B.moe_route_out(*([mem[20]] * len(B.moe_route_out._fields_)))
        big = C.c_size_t(c.get("workspace_bytes", 1 << 45))
        launches.clear()
        fail[0] = c.get("fail", -1)
        if c["entry"] == "route":
            st = L.moe_route(b, p(0), T, p(1), None, thr, full, C.byref(route), p(30), big, None)
        elif c["entry"] == "route_static":
            st = L.moe_route_static(b, p(0), T, p(1), None, thr, full, C.byref(route), None)
        elif c["entry"] == "forward":
            st = L.moe_forward(b, p(0), T, p(1), None, w(4), w(8), shared, thr, full,
                               C.byref(route) if c.get("own_route") else None, p(2), p(30), big, None)
        elif c["entry"] == "build":
            st = L.moe_build_united(b, w(4), w(8), p(0), T, p(2), p(30), big, None)
        elif c["entry"] == "distill":
            st = L.moe_distill_united(b, w(4), w(8), p(0), T, c["steps"], C.c_float(1e-3), p(2), p(30), big, None)
        else:
            raise ValueError(c["entry"])
        out.append({"status": st, "launches": list(launches)})
    json.dump(out, sys.stdout)


if __name__ == "__main__":
    _main()
