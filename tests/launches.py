"""Which kernels a call of the library launches, with which grids, found without a GPU.

launches_of(calls) runs the calls in a process of its own in which launch_recorder.c stands in for the HIP runtime:
every launch is written down instead of enqueued, device pointers are numbers that nothing dereferences.  A call is a
dict: op "forward" (fields of alora_dims, optionally rope: with rotation tables, replays: recorded and replayed, errors: a HIP error that an earlier call of the program left, and one that every
launch fails with (then: what the library reports, and what is left), timed: the shortest host time of so many
classifications and calls, tuning_during: a tuning override that arrives in the middle of the
call, between the library's two profiling events) or op "attention" (fields of alora_attn_dims and the entry point, optionally give: the workspace's size instead of the one asked for)."""
import ctypes
import json
import os
import re
import subprocess
import sys
import tempfile
import time

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


class _Launch(ctypes.Structure):
    _fields_ = [("name", ctypes.c_char * 512), ("grid", ctypes.c_uint32 * 3), ("block", ctypes.c_uint32 * 3),
                ("arg1", ctypes.c_int32), ("arg2", ctypes.c_int32)]


def launches_of(calls):
    """Per call: {"status", "workspace", "launches": [{"kernel", "ints" (of its template arguments; "contexts": of the per-row reader), "grid", "block", "args"}]}."""
    with tempfile.TemporaryDirectory() as tmp:
        rec = os.path.join(tmp, "librec.so")
        subprocess.run(["gcc", "-O1", "-w", "-shared", "-fPIC", "-o", rec, os.path.join(ROOT, "tests", "launch_recorder.c")], check=True)
        r = subprocess.run([sys.executable, os.path.abspath(__file__), rec], input=json.dumps(calls), capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stderr[-3000:]
    return json.loads(r.stdout)


def _main(rec_path):
    sys.path.insert(0, ROOT)
    rec = ctypes.CDLL(rec_path, ctypes.RTLD_GLOBAL)   # ahead of the library: its HIP calls bind here
    from paper_2512_17910_amd import binding as ab
    L = ctypes.CDLL(ab.LIB_PATH)
    rec.rec_get.restype = ctypes.POINTER(_Launch)
    P = ctypes.c_void_p(0x100000)
    HOOK = ctypes.CFUNCTYPE(None)
    out = []
    for c in json.load(sys.stdin):
        rec.rec_reset()
        rec.rec_set_error(*c.get("errors", (0, 0)))
        ws = ctypes.c_size_t(0)
        if c["op"] == "forward":
            d = ab.AloraDims(**{k: v for k, v in c.items() if k in dict(ab.AloraDims._fields_)})
            d.token_seg_ids = d.token_positions = P.value
            s = L.alora_qkv_workspace_bytes(ctypes.byref(d), ctypes.byref(ws))
            tab = (ctypes.c_void_p * max(1, d.n_adapters))(*[P.value] * d.n_adapters)
            hook = None
            if c.get("tuning_during"):
                assert L.alora_qkv_profile_begin(1) == 0
                hook = HOOK(lambda: L.alora_qkv_set_tuning(*c["tuning_during"]) and None)
                rec.rec_on_event(hook)
            if s == 0:
                if c.get("rope"):
                    ex = ab.AloraExtras(None, None, 0, P.value, P.value, 1)
                    s = L.alora_qkv_forward_ex(P, P, P, P, tab, tab, P, P, P, P, ctypes.c_int(16), ctypes.byref(d), ctypes.byref(ex), P, ws, None)
                else:
                    s = L.alora_qkv_forward(P, P, P, P, tab, tab, P, P, P, P, ctypes.c_int(16), ctypes.byref(d), P, ws, None)
            if c.get("replays"):     # the same call recorded, then replayed that many times
                assert s == 0
                rec.rec_reset()
                g = ctypes.c_void_p(None)
                s = L.alora_qkv_graph_create(P, P, P, P, tab, tab, P, P, P, P, ctypes.c_int(16), ctypes.byref(d), None, P, ws, ctypes.byref(g))
                assert rec.rec_count() == 0
                for _ in range(c["replays"]):
                    s = s or L.alora_qkv_graph_launch(g, None)
                L.alora_qkv_graph_destroy(g)
            host_us = []
            for _ in range(c.get("timed", 0)):
                rec.rec_reset()
                t = time.perf_counter()
                s = s or L.alora_qkv_classify_group(P, P, ctypes.byref(d), P, ws, None)
                s = s or L.alora_qkv_forward(P, P, P, P, tab, tab, P, P, P, P, ctypes.c_int(16), ctypes.byref(d), P, ws, None)
                host_us.append((time.perf_counter() - t) * 1e6)
            if hook:
                rec.rec_on_event(HOOK(0))
                L.alora_qkv_set_tuning(0, 0)
                L.alora_qkv_profile_end(None, None)
        else:
            d = ab.AloraAttnDims(**{k: v for k, v in c.items() if k in dict(ab.AloraAttnDims._fields_)})
            split = c["entry"].endswith("_split")
            s = getattr(L, c["entry"][:-6] + "_workspace_bytes")(ctypes.byref(d), ctypes.byref(ws)) if split else 0
            if s == 0:
                s = getattr(L, c["entry"])(P, P, P, P, P, P, P, ctypes.byref(d), *((P, ctypes.c_size_t(c.get("give", ws.value))) if split else ()), None)
        launches = []
        for i in range(rec.rec_count()):
            r = rec.rec_get(i).contents
            name = r.name.decode()
            m = re.search(r"N5alora(\d+)", name)
            launches.append({"kernel": name[m.end():m.end() + int(m.group(1))], "ints": [int(v) for v in re.findall(r"L[ib](\d+)E", name)],
                             "grid": list(r.grid), "block": list(r.block), "args": [r.arg1, r.arg2],
                             **{"contexts": int(v) for v in re.findall(r"ContextsE(\d)E", name)}})
        out.append({"status": s, "workspace": ws.value, "launches": launches, **({"host_us": min(host_us)} if c.get("timed") else {}),
                    **({"errors": [L.alora_last_hip_error(), rec.rec_error()]} if "errors" in c else {})})
    json.dump(out, sys.stdout)


if __name__ == "__main__":
    _main(sys.argv[1])
