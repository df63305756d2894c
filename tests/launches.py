"""What the library launches for a call, seen from the host: its calls into the HIP runtime are answered by
tests/hip_recorder.c, in a process of their own.  No GPU is touched and no kernel runs.

    launches([("specvlm_score", dict(n_text=64, ...), device_error, attribute_error)], directory) -> [(status, [(kernel, grid, block, lds)])]

With words=True each launch has a fifth item, the first 32 words of the kernel's first argument.

Arguments go by the names of include/specvlm.h; one that is not given is 0, a pointer None.  Pointers are made-up
addresses: nothing reads them."""
import ctypes as C
import json
import os
import re
import subprocess
import sys

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
AT = 1 << 20                                    # an address that is aligned to whatever a call asks for
TYPES = {"int": C.c_int, "int64_t": C.c_int64, "size_t": C.c_size_t, "float": C.c_float, "uint64_t": C.c_uint64}


def prototypes():
    header = open(os.path.join(ROOT, "include", "specvlm.h")).read()
    header = re.sub(r"/\*.*?\*/", "", header, flags=re.S)
    out = {}
    for ret, name, args in re.findall(r"^(size_t|int)\s+(specvlm_\w+)\(([^)]*)\);", header, flags=re.M | re.S):
        params = []
        for a in args.replace("\n", " ").split(","):
            m = re.match(r"\s*(?:const\s+)?(\w+)(\s*\*\s*|\s+)(\w+)\s*$", a)
            if m:
                params.append((m[3], C.c_void_p if "*" in m[2] else TYPES[m[1]]))
        out[name] = (TYPES[ret], params)
    return out


class Launch(C.Structure):
    _fields_ = [("name", C.c_char_p), ("grid", C.c_uint * 3), ("block", C.c_uint * 3), ("lds", C.c_size_t), ("words", C.c_int * 32)]


def _serve(recorder, library):
    rec = C.CDLL(recorder, mode=C.RTLD_GLOBAL)
    lib, protos, answers = C.CDLL(library), prototypes(), []
    taken = (Launch * 256)()
    for name, args, device_error, attribute_error in json.load(sys.stdin):
        ret, params = protos[name]
        unknown = set(args) - {n for n, _ in params}
        assert not unknown, unknown
        f = getattr(lib, name)
        f.restype, f.argtypes = ret, [t for _, t in params]
        rec.recorder_errors(device_error, attribute_error)
        status = f(*[args.get(n, None if t is C.c_void_p else 0) for n, t in params])
        n = rec.recorder_take(taken)
        answers.append([status, [[l.name.decode(), list(l.grid), list(l.block), l.lds, list(l.words)] for l in taken[:n]]])
    json.dump(answers, sys.stdout)


def launches(calls, directory, words=False):
    """calls: [(function, arguments[, device error[, attribute error]])]"""
    recorder = os.path.join(str(directory), "recorder.so")
    subprocess.run(["gcc", "-O1", "-w", "-shared", "-fPIC", "-o", recorder, os.path.join(ROOT, "tests", "hip_recorder.c")], check=True)
    library = os.path.join(ROOT, "paper_2508_16201_amd", "libspecvlm.so")
    if not os.path.exists(library):
        from paper_2508_16201_amd import build
        build.build()
    full = [(*c, *(0, 0))[:4] for c in calls]
    res = subprocess.run([sys.executable, os.path.abspath(__file__), recorder, library], input=json.dumps(full), capture_output=True,
                         text=True, timeout=120)
    assert res.returncode == 0, (res.returncode, res.stderr[-2000:])
    answers = json.loads(res.stdout)
    names = sorted({l[0] for _, ls in answers for l in ls})
    plain = subprocess.run(["c++filt", *names], capture_output=True, text=True, check=True).stdout.splitlines() if names else []
    short = {n: re.sub(r"\(specvlm::.*|void |specvlm::", "", p) for n, p in zip(names, plain)}
    return [(status, [(short[n], tuple(grid), tuple(block), lds, w)[:5 if words else 4] for n, grid, block, lds, w in ls]) for status, ls in answers]


if __name__ == "__main__":
    _serve(*sys.argv[1:])
