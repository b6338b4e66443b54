"""Which kernels a call launches, without a GPU: the library's dispatch runs
on the host, with launch_recorder.c in place of the HIP runtime."""
import collections
import json
import os
import shutil
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
LIB = os.path.join(os.path.dirname(HERE), "paper_2606_06751_amd", "libstagefrontier.so")

LLVM = "/opt/rocm/llvm/bin/"
Launch = collections.namedtuple("Launch", "name grid block lds")


def build_recorder(folder) -> str:
    cc = shutil.which("gcc") or shutil.which("cc")
    if cc is None:
        import pytest
        pytest.skip("no C compiler")
    so = os.path.join(str(folder), "librecorder.so")
    subprocess.run([cc, "-O1", "-shared", "-fPIC", "-o", so, os.path.join(HERE, "launch_recorder.c")], check=True)
    return so


def _args(call, R, S, T, window):
    dims = [("l", T), ("i", R), ("i", S)]
    n_in = {"sf_exposure_gain": 2, "sf_window_summary": 2, "sf_window_lead_exposed": 2}.get(call, 1)
    n_out = {"sf_frontier": 2, "sf_frontier_checked": 3, "sf_frontier_evidence": 6, "sf_frontier_lag": 2,
             "sf_rank_spread": 2, "sf_window_median": 1, "sf_exposure_gain": 4, "sf_window_summary": 3,
             "sf_frontier_summary": 5, "sf_window_lead_exposed": 2}[call]
    if call not in ("sf_frontier", "sf_frontier_checked", "sf_frontier_evidence", "sf_frontier_lag"):
        dims = dims + [("l", window)]
    ptr = ["p%d" % i for i in range(n_in + n_out)]
    return ptr[:n_in] + dims + ptr[n_in:] + [("l", 0)]


def launches(recorder, cases, lib=LIB):
    """Per case (call, R, S, T, window): its list of launches, the kernels'
    names demangled."""
    req = [[c[0], _args(*c)] for c in cases]
    p = subprocess.run([sys.executable, os.path.join(HERE, "launch_probe.py"), recorder, lib],
                       input=json.dumps(req), capture_output=True, text=True, check=True)
    res = json.loads(p.stdout)
    names = sorted({l[0] for _, ls in res for l in ls})
    plain = subprocess.run(["c++filt"] + names, capture_output=True, text=True, check=True).stdout.split("\n")
    short = {n: d.replace("void ", "").replace("sfk::", "").split("(")[0] for n, d in zip(names, plain)}
    for c, (rc, _) in zip(cases, res):
        assert rc == 0, (c, rc)
    return [[Launch(short[n], g, b, l) for n, g, b, l in ls] for _, ls in res]


def spilled_vgprs(folder, lib=LIB):
    """Spilled vector registers of every kernel in the built library, from the
    metadata of its code objects."""
    data = open(lib, "rb").read()
    out, at = {}, data.find(b"\x7fELF", 4)
    while at >= 0:
        if int.from_bytes(data[at + 18:at + 20], "little") == 224:  # an AMDGPU code object
            end = data.find(b"\x7fELF", at + 4)
            path = os.path.join(str(folder), "object.elf")
            with open(path, "wb") as fh:
                fh.write(data[at:end if end > 0 else len(data)])
            notes = subprocess.run([LLVM + "llvm-readelf", "--notes", path], capture_output=True, text=True).stdout
            name = None
            for line in notes.split("\n"):
                key, _, value = line.strip().lstrip("- ").partition(":")
                if key == ".name" and value.strip().startswith("_Z"):
                    name = value.strip()
                elif key == ".vgpr_spill_count" and name:
                    out[name] = int(value)
        at = data.find(b"\x7fELF", at + 4)
    plain = subprocess.run(["c++filt"] + list(out), capture_output=True, text=True, check=True).stdout.split("\n")
    return {d.replace("void ", "").replace("sfk::", "").split("(")[0]: n for d, n in zip(plain, out.values())}
