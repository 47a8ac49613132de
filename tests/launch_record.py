"""What the library launches for a call, found without a GPU: a child process loads the library on top of tests/launch_recorder.cpp
(its functions come before the HIP runtime's) and makes the calls with made-up addresses."""
import ctypes
import json
import os
import subprocess
import sys
import time
import types

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)


def record(calls, tmp_path):
    """One dict per call: rc, bytes (of its workspace), launches, a list of (kernel, grid, block, dynamic LDS bytes, cap on them), and us, the shortest time
    that the entry point took of the host.  A call is a dict of `entry`, its sizes (see the functions below), and optionally `device` (the current device),
    `fail_attributes` (the runtime refuses to raise a cap) and `repeat`."""
    lib = os.path.join(str(tmp_path), "launch_recorder.so")
    if not os.path.exists(lib):
        subprocess.run(["g++", "-O1", "-std=c++17", "-shared", "-fPIC", os.path.join(HERE, "launch_recorder.cpp"), "-o", lib], check=True)
    r = subprocess.run([sys.executable, os.path.abspath(__file__), lib], input=json.dumps(calls), capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stderr[-2000:]
    return json.loads(r.stdout)


# ---- the child
class _Tensor:
    """An address; 256-byte aligned, `skew` bytes off where alignment is the point."""
    is_cuda = True
    _next = 1 << 40

    def __init__(self, n_bytes=1 << 30, skew=0):
        self.addr, self.n = _Tensor._next + skew, n_bytes
        _Tensor._next += 1 << 32

    def is_contiguous(self):
        return True

    def data_ptr(self):
        return self.addr

    def numel(self):
        return self.n

    def element_size(self):
        return 1


def _layer_desc(B, c):
    return B.LayerDesc(B.vq_desc(c.get("dtype", "bf16"), c["d"], c["groups"], c["words"]), _attn_desc(B, c))


def _attn_desc(B, c):
    n_n = c["n_nonlocal"]
    return B.attn_desc(c.get("dtype", "bf16"), c["hq"], c["hkv"], c["dh"], c.get("cls", 0), c["n_local"], n_n, c.get("causal", False),
                       c.get("before", n_n if c.get("causal") else 0))


def _layer(B, c, t):
    desc = _layer_desc(B, c)
    b = [t() if c.get("bias") else None for _ in range(4)]
    n = B.astra_layer_workspace_bytes(desc)
    if c["entry"] == "preprojected":
        B.astra_layer_forward_preprojected(desc, t(), t(), None, *[t() for _ in range(8)], *b, t(), t(), _Tensor(n))
    else:
        B.astra_layer_forward(desc, t(), t(), t(), t(), *[t() for _ in range(4)], *b, t(), t(), _Tensor(n))
    return n


def _block(B, c, t):
    desc = B.block_desc(_layer_desc(B, c), c["norm"], c["mlp"], c["dff"], 1e-5, c.get("rope", 0.0))
    names = ["codebook", "cnorm", "wq", "wk", "wv", "wo", "w1", "w2", "norm1_gain", "norm2_gain"]
    if c.get("bias"):
        names += ["bq", "bk", "bv", "bo", "b1", "b2"]
    n = B.astra_block_workspace_bytes(desc)
    B.astra_block_forward(desc, B.block_weights(**{k: t() for k in names}), t(), t(), None, t(), t(), None, _Tensor(n))
    return n


def _stack(B, c, t):
    desc = B.block_desc(_layer_desc(B, c), c["norm"], c["mlp"], c["dff"], 1e-5, c.get("rope", 0.0))
    names = ["codebook", "cnorm", "wq", "wk", "wv", "wo", "w1", "w2", "norm1_gain", "norm2_gain"]
    n, blocks = B.astra_block_workspace_bytes(desc), range(c["layers"])
    B.astra_stack_forward(desc, [B.block_weights(**{k: t() for k in names}) for _ in blocks], t(), [t() for _ in blocks], None, t(), [t() for _ in blocks],
                          _Tensor(n))
    return n


def _kv(B, c, t):
    desc = B.LayerKvDesc(B.vq_desc("bf16", c["hkv"] * c["dh"], c["groups"], c["words"]), _attn_desc(B, c), c["d"])
    n = B.astra_layer_kv_workspace_bytes(desc)
    B.astra_layer_forward_kv(desc, t(), t(), t(), None, t(), t(), t(), t(), *[t() for _ in range(4)], *[None] * 4, t(), t(), t(), t(), t(),
                             _Tensor(n))
    return n


def _project(B, c, t):
    B.astra_vq_project_codebook(B.vq_desc(c.get("dtype", "bf16"), c["k"], 1, c["m"]), t(), t(), c["n"], t())
    return 0


def _step(B, c, t):
    desc = B.DecodeDesc(B.vq_desc(c.get("dtype", "bf16"), c["hkv"] * c["dh"], c["groups"], c["words"]), c["hq"], c["hkv"], c["dh"], c["n_local"],
                        c["n_nonlocal"], 0.0)
    n = B.astra_decode_attention_workspace_bytes(desc)
    B.astra_decode_attention(desc, t(), t(), t(), t(), t(), None, t(), t(), t(), None, _Tensor(n))
    return n


def _stats(B, c, t):
    desc = B.vq_desc(c.get("dtype", "bf16"), c["groups"] * c["dg"], c["groups"], c["words"])
    n = B.astra_codebook_stats_workspace_bytes(desc, c["tokens"])
    B.astra_codebook_stats(desc, t(), t(), c["tokens"], t(), t(), t(), t(), _Tensor(n))
    return n


def _update(B, c, t):
    desc = B.vq_desc(c.get("dtype", "bf16"), c["groups"] * c["dg"], c["groups"], c["words"])
    B.astra_codebook_update(desc, t(), t(), 0.9, t(), t(), t(), _Tensor(skew=c.get("skew", 0)))
    return 0


def _encode(B, c, t):
    desc = B.vq_desc(c.get("dtype", "bf16"), c["d"], c["groups"], c["words"])
    n = B.astra_vq_encode_workspace_bytes(desc, c["tokens"])
    x, codebook, cnorm = (t(skew=c.get("skew", {}).get(a, 0)) for a in ("x", "codebook", "cnorm"))
    B.astra_vq_encode_ws(desc, x, c["tokens"], codebook, cnorm, t(), _Tensor(n))
    return n


def _main(recorder):
    rec = ctypes.CDLL(recorder, mode=ctypes.RTLD_GLOBAL)      # before the library: its symbols resolve to these first
    rec.rec_name.restype = ctypes.c_char_p
    sys.modules["torch"] = types.ModuleType("torch")          # no other HIP runtime in this process
    sys.path.insert(0, os.environ.get("LAUNCH_RECORD_TREE", ROOT))
    from paper_2505_19342_amd import binding as B
    B.load(build_if_missing=False)
    B._stream = lambda: None
    entries = {"layer": _layer, "preprojected": _layer, "block": _block, "stack": _stack, "kv": _kv, "project": _project, "step": _step, "stats": _stats, "update": _update, "encode": _encode}
    plain = {n: getattr(B, n) for n in ("astra_layer_forward", "astra_layer_forward_kv", "astra_block_forward", "astra_stack_forward")}
    spent = []

    def timed(f):
        def g(*a):
            t = time.perf_counter()
            f(*a)
            spent.append(time.perf_counter() - t)
        return g
    for n, f in plain.items():
        setattr(B, n, timed(f))
    out = []
    for c in json.load(sys.stdin):
        spent.clear()
        rc, n = "ok", 0
        try:
            for _ in range(c.get("repeat", 1)):
                rec.rec_reset(c.get("device", 0), int(c.get("fail_attributes", False)))
                n = entries[c["entry"]](B, c, _Tensor)
        except B.AstraError as e:
            rc = str(e)
        launches = []
        for i in range(rec.rec_count()):
            grid, block = (ctypes.c_uint32 * 3)(), (ctypes.c_uint32 * 3)()
            lds, cap = ctypes.c_size_t(), ctypes.c_size_t()
            rec.rec_shape(i, grid, block, ctypes.byref(lds), ctypes.byref(cap))
            name = rec.rec_name(i).decode().replace("(anonymous namespace)::", "").replace("void ", "").replace("astra::", "").split("(")[0]
            launches.append((name, list(grid), list(block), lds.value, cap.value))
        out.append({"rc": rc, "bytes": n, "launches": launches, "us": min(spent, default=0.0) * 1e6})
    json.dump(out, sys.stdout)


if __name__ == "__main__":
    _main(sys.argv[1])
