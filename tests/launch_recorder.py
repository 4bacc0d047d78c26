"""What the library launches for a call, without a GPU: the calls of clasp.h on made-up device addresses against the recording
runtime of hip_recorder.cpp. Imports neither torch nor the package's binding: it has to run in a process in which nothing
else has loaded the HIP runtime (tests run it as `python launch_recorder.py <recorder.so> <library.so>` with a list of jobs on stdin
and read the launches from stdout)."""
import ctypes as C
import json
import sys

ADDR = 0x100000000  # made-up device addresses, 256-byte aligned, never dereferenced


class Config(C.Structure):
    _fields_ = [(n, C.c_int32) for n in ("n_layers", "d_model", "n_heads", "n_kv_heads", "head_dim", "d_ffn", "vocab",
                                         "max_seq", "max_rows", "dtype")] + [("rms_eps", C.c_float), ("rope_base", C.c_float)]


class Weights(C.Structure):
    _fields_ = [(n, C.c_void_p) for n in ("embed", "lm_head", "final_norm", "attn_norm", "mlp_norm", "wq", "wk", "wv", "wo",
                                          "w_gate_up", "w_down")]


def call(lib, ctx, cfg, name, *a):
    p = C.c_void_p(ADDR)
    mask = (C.c_uint8 * cfg.n_layers)()
    f = C.c_float
    if name == "verify":  # rows, position
        return lib.clasp_verify_forward(ctx, p, a[0], a[1], p, p, p, p, None)
    if name == "dp":  # position, budget
        return lib.clasp_dp_select(ctx, p, C.c_size_t(cfg.d_model), a[0], a[1], p, None, None, None, None)
    if name == "draft":  # position
        return lib.clasp_draft_sample(ctx, mask, p, a[0], f(1.0), p, p, p, None)
    if name == "accept":  # drafts
        return lib.clasp_spec_accept(ctx, p, p, C.c_size_t(cfg.vocab), p, a[0], f(1.0), p, p, p, p, None)
    if name == "kv_load":  # positions
        return lib.clasp_kv_load(ctx, 0, p, p, a[0], None)
    if name == "kv_read":  # first position, positions
        return lib.clasp_kv_read(ctx, 0, a[0], a[1], p, p, None)
    if name == "prefill":  # rows, position, rows per pass
        need = lib.clasp_prefill_workspace_bytes(C.byref(cfg), a[2])
        return lib.clasp_prefill(ctx, p, a[0], a[1], a[2], p, C.c_size_t(need), None)
    raise ValueError(name)


def main():
    rec = C.CDLL(sys.argv[1], mode=C.RTLD_GLOBAL)
    lib = C.CDLL(sys.argv[2])
    rec.recorder_log.restype = rec.recorder_kernels.restype = C.c_char_p
    lib.clasp_workspace_bytes.restype = lib.clasp_prefill_workspace_bytes.restype = C.c_size_t
    out = []
    for job in json.load(sys.stdin):  # {"config": [...10 ints], "device": d, "calls": [[name, args..], ..]}
        rec.recorder_set_device(job.get("device", 0))
        cfg = Config(*job["config"], 1e-5, 10000.0)
        L = cfg.n_layers
        ptrs = (C.c_void_p * L)(*[ADDR] * L)
        w = Weights(ADDR, ADDR, ADDR, *[C.cast(ptrs, C.c_void_p)] * 8)
        ctx = C.c_void_p()
        size = lib.clasp_workspace_bytes(C.byref(cfg))
        assert size, "configuration refused"
        rc = lib.clasp_create(C.byref(cfg), C.byref(w), C.c_void_p(ADDR), C.c_size_t(size), C.c_void_p(ADDR), C.c_void_p(ADDR),
                              C.byref(ctx))
        assert rc == 0, rc
        for c in job["calls"]:
            rec.recorder_clear()
            rc = call(lib, ctx, cfg, *c)
            rows = [line.split("\t") for line in rec.recorder_log().decode().splitlines()]
            out.append({"call": c, "rc": rc, "launches": [
                {"kernel": r[0], "grid": [int(x) for x in r[1:4]], "threads": int(r[4]), "lds": int(r[5]), "device": int(r[6]),
                 "lds_allowed": r[7] == "1"} for r in rows]})
        lib.clasp_destroy(ctx)
    json.dump({"calls": out, "kernels": rec.recorder_kernels().decode().splitlines()}, sys.stdout)


if __name__ == "__main__":
    main()
