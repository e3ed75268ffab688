"""Which kernels a call of the library launches, on a machine without a GPU.

run(calls) starts a process of its own in which libvq.so finds launch_log.cpp in place of the HIP runtime, makes the calls there and returns for
each its status, the workspace that was asked for and the launches.  A call is a dict: "entry" (an entry point's name without vq_), "layer" (sizes of
a descriptor; pointers and strides are made up), "rows", "pitch" and "x" (columns from one row of activations to the next, address of the
first; both have defaults), "workspace" (bytes; None: none; "asked": what the library asks for; "lent": what
the package lends gemv() of its own accord; "least": gemm() on a card without room for what the library asks for), "asked_for_rows" (whose size that is; default: "rows").
"""
import ctypes
import json
import os
import subprocess
import sys
import tempfile

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
WORKSPACE = 1 << 40                      # made-up addresses: nothing is read or written
X, Y = 1 << 41, 1 << 42


def run(calls, lib=None, switches=None):
    with tempfile.TemporaryDirectory() as folder:
        shim = os.path.join(folder, "launch_log.so")
        subprocess.check_call(["g++", "-O1", "-std=c++17", "-shared", "-fPIC", os.path.join(HERE, "launch_log.cpp"), "-o", shim])
        env = dict(os.environ, VQ_SWITCHES=switches or "")
        done = subprocess.run([sys.executable, os.path.abspath(__file__), shim, lib or ""], input=json.dumps(calls), stdout=subprocess.PIPE, text=True,
                              cwd=ROOT, env=env)
    assert done.returncode == 0
    return json.loads(done.stdout)


def _bits(k):
    return max(1, (k - 1).bit_length())


def _descriptor(vq, layer):
    d = dict(v=6, k=4096, k_res=0, n_outlier_cols=0, v_out=4, k_out=4096, group_vectors=0, orientation=0, col_perm=False)
    d.update(layer)
    down, main = d["orientation"] == 1, d["in_features"] - d["n_outlier_cols"]

    def stride(count, k):
        return (count * _bits(k) + 127) // 128 * 16
    vectors = main if down else -(-main // d["v"])
    outliers = d["n_outlier_cols"] if down else d["n_outlier_cols"] // d["v_out"]
    at = 1 << 43
    return vq.vq_layer_desc(ctypes.sizeof(vq.vq_layer_desc), d["out_features"], d["in_features"], d["v"], d["k"], d["k_res"], d["n_outlier_cols"],
                            d["v_out"], d["k_out"], at, at, at, at, stride(vectors, d["k"]), at, stride(vectors, d["k_res"] or 2), at, stride(outliers, d["k_out"]),
                            at, at, d["group_vectors"], d["orientation"], at if d["col_perm"] else None)


def _main(shim, lib):
    log = ctypes.CDLL(shim, mode=ctypes.RTLD_GLOBAL)
    log.launch_log.restype = ctypes.c_char_p
    sys.modules["torch"] = None          # (it would bring the HIP runtime itself)
    sys.path.insert(0, ROOT)
    import paper_2409_17066_amd as vq
    if lib:
        vq.LIB_PATH = lib
    vq.load()
    out = []
    for call in json.load(sys.stdin):
        d, rows, entry = _descriptor(vq, call["layer"]), call["rows"], call["entry"]
        n, m = d.in_features, d.out_features
        gemv = entry.startswith("gemv")
        size = vq.vq_gemv_workspace_bytes if gemv else vq.vq_gemm_default_workspace_bytes if entry == "gemm_default" else vq.vq_gemm_fast_workspace_bytes
        asked = size(d, call.get("asked_for_rows", rows))
        pitch = call.get("pitch", n + (n & 1) if gemv else (n + 7) // 8 * 8)
        bytes_ = call.get("workspace")
        bytes_ = asked if bytes_ == "asked" else vq.load().vq_lend_gemv_bytes(ctypes.byref(d), rows) if bytes_ == "lent" else bytes_
        bytes_ = vq.load().vq_lend_gemm_least_bytes(ctypes.byref(d), rows) if bytes_ == "least" else bytes_
        x = call.get("x", X)
        log.launch_log_clear()
        if entry in ("gemv", "gemv_static_workspace"):
            rc = getattr(vq, "vq_" + entry)(d, x, pitch, rows, Y, m)
        else:
            f = {"gemv_with_workspace": vq.vq_gemv_with_workspace, "gemm": vq.vq_gemm, "gemm_default": vq.vq_gemm_default}[entry]
            rc = f(d, x, pitch, rows, Y, m, WORKSPACE if bytes_ else None, bytes_ or 0)
        launches = []
        for line in log.launch_log().decode().splitlines():
            name, grid, threads, lds, words = line.split("|")
            launches.append(dict(name=name.replace("vq::", "").split("void ")[-1], grid=[int(g) for g in grid.split()], threads=int(threads), lds=int(lds),
                                 words=[int(w) for w in words.split()]))
        out.append(dict(status=rc, asked=asked, lent=bytes_ or 0, launches=launches))
    json.dump(out, sys.stdout)


if __name__ == "__main__":
    _main(sys.argv[1], sys.argv[2])
