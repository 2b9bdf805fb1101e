"""The library's host code under a HIP runtime that computes nothing (fake_hip.cpp), in a process of its own: what
hgemm_plan and hgemm_run_static decide, allocate and launch, on a machine without a GPU.

    ask([{"M": 8, "N": 8, "K": 8, ...}, ...]) -> one dict per question: status, description, workspace bytes, reported workgroups and log of
    hgemm_plan (hgemm_plan_override, where a spec is given) + hgemm_run (and of hgemm_run_many, where operand sets are given), and status and log of hgemm_run_static, on
    operands at the addresses asked for."""
import ctypes
import json
import os
import subprocess
import sys
import tempfile

HERE = os.path.dirname(os.path.abspath(__file__))
LIB = os.path.join(os.path.dirname(HERE), "paper_2512_02551_amd", "libhgemm.so")
BASE = 1 << 36          # an aligned address; nothing is ever read from it


def ask(questions):
    with tempfile.TemporaryDirectory() as tmp:
        so = os.path.join(tmp, "libfake_hip.so")
        subprocess.run(["g++", "-O1", "-shared", "-fPIC", "-I/opt/rocm/include", os.path.join(HERE, "fake_hip.cpp"), "-o", so], check=True)
        res = subprocess.run([sys.executable, os.path.abspath(__file__), so], input=json.dumps(questions), stdout=subprocess.PIPE, text=True, check=True)
    return json.loads(res.stdout)


def _answer(fake, lib, q):
    class Layouts(ctypes.Structure):
        _fields_ = [("a", ctypes.c_int), ("b", ctypes.c_int), ("c", ctypes.c_int),
                    ("lda", ctypes.c_int64), ("ldb", ctypes.c_int64), ("ldc", ctypes.c_int64)]

    def log():
        return fake.fake_take_log().decode().splitlines()

    i64, vp = ctypes.c_int64, ctypes.c_void_p
    lay = Layouts(0, int(q.get("tn", False)), 0, q.get("lda", 0), q.get("ldb", 0), q.get("ldc", 0))
    dims = [i64(q[d]) for d in "MNK"]
    at = [vp(q.get(p, BASE)) for p in "ABC"]
    fake.fake_device_memory(ctypes.c_size_t(q.get("memory", 1 << 40)))
    plan = vp()
    log()
    spec = [q["spec"].encode()] if "spec" in q else []
    r = {"plan": (lib.hgemm_plan_override if spec else lib.hgemm_plan)(ctypes.byref(plan), *dims, ctypes.byref(lay), *spec), "plan_log": log()}
    if r["plan"] == 0:
        text = ctypes.create_string_buffer(512)
        assert lib.hgemm_plan_describe(plan, text, ctypes.c_size_t(512)) == 0
        r["describe"], r["workspace"] = text.value.decode(), lib.hgemm_plan_workspace_bytes(plan)
        groups = i64()
        assert lib.hgemm_plan_launch_info(plan, ctypes.byref(groups), None, None) == 0
        r["workgroups"] = groups.value
        r["run"], r["run_log"] = lib.hgemm_run(plan, *at, None), log()
        if "many" in q:         # (A, B, C) per operand set
            arrays = [(vp * len(q["many"]))(*column) for column in zip(*q["many"])]
            r["many"] = lib.hgemm_run_many(plan, i64(q.get("count", len(q["many"]))), i64(len(q["many"])), i64(q.get("first", 0)), *arrays, None)
            r["many_log"] = log()
        lib.hgemm_destroy(plan)
        assert fake.fake_live_bytes() == 0, "the plan's memory was not given back"
    log()
    r["static"], r["static_log"] = lib.hgemm_run_static(*dims, ctypes.byref(lay), *at, None), log()
    return r


if __name__ == "__main__":
    fake_lib = ctypes.CDLL(sys.argv[1], mode=ctypes.RTLD_GLOBAL)
    fake_lib.fake_take_log.restype = ctypes.c_char_p
    fake_lib.fake_live_bytes.restype = ctypes.c_size_t
    hgemm_lib = ctypes.CDLL(LIB)
    hgemm_lib.hgemm_plan_workspace_bytes.restype = ctypes.c_size_t
    print(json.dumps([_answer(fake_lib, hgemm_lib, q) for q in json.load(sys.stdin)]))
