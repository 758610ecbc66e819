"""Which kernels the library launches for a call, on the CPU: the calls run in a child process whose HIP launch calls are
those of launch_recorder.c, on addresses that nothing dereferences."""
import ctypes as C
import json
import os
import re
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
ADDRESS = 1 << 40       # of every operand: aligned, never read


def launches(tmp_path, calls, lds_limit_fails=False):
    """calls: [["gemm", dict(prec, M, N, K, and optionally lda, ak, ldb, bk, ldc, f32, epi)] or ["layer_bwd", cfg] or
    ["mlm", dict]].  Per call (status, [(kernel name, template arguments, (grid x, grid y)), ...])."""
    so = str(tmp_path / "recorder.so")
    subprocess.run(["gcc", "-O1", "-shared", "-fPIC", "-o", so, os.path.join(HERE, "launch_recorder.c"), "-ldl"], check=True)
    p = subprocess.run([sys.executable, os.path.abspath(__file__), so, str(int(lds_limit_fails))], input=json.dumps(calls),
                       capture_output=True, text=True, timeout=300)
    assert p.returncode == 0, p.stderr[-2000:]
    out = []
    for status, found in json.loads(p.stdout.splitlines()[-1]):
        kernels = []
        for name, gx, gy in found:
            m = re.match(r"_ZN3raf(\d+)(.*)", name)
            assert m, name
            n, rest = int(m.group(1)), m.group(2)
            args = re.match(r"I(.*?)E?Ev", rest[n:])
            values = tuple(int(v) for v in re.findall(r"L[ib](\d+)E", rest[n:])) if args else ()
            kernels.append((rest[:n], values, (gx, gy)))
        out.append((status, kernels))
    return out


def _child(so, fail):
    rec = C.CDLL(so, mode=C.RTLD_GLOBAL)
    rec.recorder_name.restype = C.c_char_p
    sys.path.insert(0, os.path.dirname(HERE))
    import paper_2303_04759_amd as raf
    lib = raf.load_library()
    answers = []
    for kind, a in json.load(sys.stdin):
        rec.recorder_reset(fail)
        if kind == "gemm":
            M, N, K, ak, bk = a["M"], a["N"], a["K"], a.get("ak", 1), a.get("bk", 1)
            status = lib.raf_op_gemm(a["prec"], M, N, K, ADDRESS, a.get("lda", K if ak else M), ak, ADDRESS,
                                     a.get("ldb", K if bk else N), bk, ADDRESS, a.get("ldc", N), a.get("f32", 0), 1.0,
                                     a.get("epi", 0), ADDRESS, ADDRESS, 0, None)
        elif kind == "layer_bwd":
            t = raf.LayerTensors()
            for name in raf.PARAM_NAMES:
                setattr(t, name, ADDRESS)
            status = lib.raf_layer_bwd(C.byref(raf.make_desc(a)), C.byref(t), ADDRESS, ADDRESS, ADDRESS, ADDRESS, ADDRESS,
                                       C.byref(t), ADDRESS, 1, None)
        else:
            raise ValueError(kind)
        n = rec.recorder_count()
        answers.append((status, [(rec.recorder_name(i).decode(), rec.recorder_grid(i, 0), rec.recorder_grid(i, 1))
                                 for i in range(n)]))
    print(json.dumps(answers))


if __name__ == "__main__":
    _child(sys.argv[1], int(sys.argv[2]))
