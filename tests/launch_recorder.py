"""Records what libsigk's host side launches, without a GPU: ``record(jobs)`` runs
the jobs in a process of its own whose HIP runtime is launch_recorder.cpp.

A job is a dict: {"call": "gram" | "pair_backward" | "plan" | "cus" | ..., ...}
(see _run); its result is {"rc": code, "events": [[what, kernel, grid, block,
lds], ...]} with kernel names shortened to ``name<args>``.  Device pointers are
addresses nothing dereferences."""
import ctypes
import importlib.util
import json
import os
import re
import subprocess
import sys
import tempfile

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
SONAME = "libamdhip64.so.7"

# Waves per CU the kernels reach on an MI355X (part of the mangled name; the
# longest match counts, 4 = one wave per SIMD otherwise)
OCCUPANCY = {"10fwd_kernelILi4ELi8E": 12, "10fwd_kernelILi4ELi16E": 8,
             "10fwd_kernelILi5ELi8E": 11, "10fwd_kernelILi5ELi16E": 8,
             "10fwd_kernelILi6ELi8E": 12, "10fwd_kernelILi6ELi16E": 8,
             "10fwd_kernelILi8ELi8E": 8, "10fwd_kernelILi8ELi16E": 7,
             "10fwd_kernelILi10ELi8E": 8, "10fwd_kernelILi10ELi16ELb0ELi64E": 8,
             "10fwd_kernelILi12ELi8ELb0ELi64E": 8,
             **{f"11team_kernelILi{p}ELi{d}E": 12 for p in (4, 5, 6) for d in (0, 8)},
             **{f"11team_kernelILi{p}ELi16E": 8 for p in (4, 5, 6, 8, 10)},
             **{f"11team_kernelILi{p}ELi{d}E": 8 for p in (8, 10) for d in (0, 8)},
             # (their forms of one wave per SIMD)
             "10fwd_kernelILi8ELi16ELb0ELi64ELb1E": 4, "10fwd_kernelILi10ELi8ELb0ELi64ELb1E": 5,
             "10fwd_kernelILi10ELi16ELb0ELi64ELb1E": 4, "10fwd_kernelILi12ELi8ELb0ELi64ELb1E": 4}


def record(jobs):
    with tempfile.TemporaryDirectory() as tmp:
        lib = os.path.join(tmp, SONAME)
        ver = os.path.join(tmp, "v.map")
        with open(ver, "w") as f:
            f.write("hip_4.2 { global: hip*; __hip*; rec_*; };\n")
        subprocess.run(["g++", "-std=c++17", "-O1", "-shared", "-fPIC", f"-Wl,-soname,{SONAME}",
                        f"-Wl,--version-script={ver}", os.path.join(HERE, "launch_recorder.cpp"),
                        "-o", lib], check=True)
        p = subprocess.run([sys.executable, os.path.abspath(__file__), lib],
                           input=json.dumps(jobs), capture_output=True, text=True, timeout=120)
    assert p.returncode == 0, p.stderr[-2000:]
    return json.loads(p.stdout)


def kernels(result):
    """Names of the launched kernels, in order."""
    return [e[1] for e in result["events"] if e[0] == "launch"]


def _short(mangled):
    m = re.match(r"_ZN(?:4sigk|\d*_GLOBAL__N_1|12_GLOBAL__N_1)?(\d+)", mangled)
    if not m:
        return mangled
    n, rest = int(m.group(1)), mangled[m.end():]
    args = re.match(r"I((?:L[ib]\d+E)+)E", rest[n:])
    vals = re.findall(r"L[ib](\d+)E", args.group(1)) if args else []
    return rest[:n] + (f"<{','.join(vals)}>" if vals else "")


def _main():
    rec = ctypes.CDLL(sys.argv[1], mode=ctypes.RTLD_GLOBAL)
    rec.rec_what.restype = rec.rec_name.restype = ctypes.c_char_p
    for part, n in OCCUPANCY.items():
        rec.rec_set_occupancy(part.encode(), n)
    spec = importlib.util.spec_from_file_location(
        "sigk_binding", os.path.join(ROOT, "paper_2502_20392_amd", "_lib.py"))
    binding = importlib.util.module_from_spec(spec)
    spec.loader.exec_module(binding)
    out = []
    for job in json.load(sys.stdin):
        rec.rec_clear()
        res = _run(job, rec, binding)
        ev = []
        for i in range(rec.rec_count()):
            sz = (ctypes.c_longlong * 3)()
            rec.rec_sizes(i, sz)
            ev.append([rec.rec_what(i).decode(), _short(rec.rec_name(i).decode()), *sz])
        res["events"] = ev
        out.append(res)
    print(json.dumps(out))


def _run(job, rec, binding):
    if job["call"] == "cus":
        rec.rec_set_cus(job["n"])
        return {"rc": 0}
    lib = binding.load()
    dev = ctypes.c_void_p(1 << 40)
    big = ctypes.c_size_t(1 << 50)
    o = binding.make_opts(job.get("order", 12), grid=job.get("grid", 0), tile=job.get("tile", 0),
                          field=job.get("field", False), square=job.get("square", False))
    if job["call"] == "gram":
        nx, lx, d = job["nx"], job["lx"], job["d"]
        ny, ly = job.get("ny", nx), job.get("ly", lx)
        sym = int("ny" not in job)
        return {"rc": lib.sigk_gram(dev, nx, dev, ny, lx, ly, d, sym, ctypes.byref(o), dev, dev,
                                    big, None)}
    if job["call"] == "pair_backward":
        lx, ly, d = job["lx"], job["ly"], job["d"]
        rows, cols = job.get("rows", 0), job.get("cols", 0)
        nb = ctypes.c_size_t()
        rc = lib.sigk_pair_backward_workspace_size(lx, ly, d, rows, cols, ctypes.byref(o),
                                                   ctypes.byref(nb))
        if rc or job.get("ws") == 0:
            return {"rc": rc, "bytes": nb.value}
        ws = ctypes.c_size_t(job.get("ws") or nb.value)
        rc = lib.sigk_pair_backward(dev, lx, dev, ly, d, dev, rows, cols, ctypes.byref(o), dev,
                                    dev, dev, dev, ws, None)
        return {"rc": rc, "bytes": nb.value}
    if job["call"] == "plan":
        lens, d = job["lens"], job["d"]
        off = (ctypes.c_int64 * (len(lens) + 1))(*[sum(lens[:i]) for i in range(len(lens) + 1)])
        prs = [v for p in job["pairs"] for v in p]
        pairs = (ctypes.c_int32 * len(prs))(*prs)
        h = ctypes.c_void_p()
        rc = lib.sigk_plan_ragged(off, len(lens), d, pairs, len(job["pairs"]), ctypes.byref(o),
                                  ctypes.byref(h))
        for step in job["steps"]:
            rc = rc or {"upload": lambda: lib.sigk_plan_upload(h, dev, big, None),
                        "run": lambda: lib.sigk_plan_run(h, dev, dev, dev, big, None),
                        "backward": lambda: lib.sigk_plan_backward(h, dev, dev, dev, dev, big,
                                                                   None)}[step]()
        lib.sigk_plan_destroy(h)
        return {"rc": rc}
    raise ValueError(job["call"])


if __name__ == "__main__":
    _main()
