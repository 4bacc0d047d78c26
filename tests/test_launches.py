"""What the library's host side launches, looked at without a GPU (launch_recorder.py)."""
import json
import os
import subprocess
import sys

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
F32, BF16 = 0, 1


@pytest.fixture(scope="module")
def recorder(tmp_path_factory):
    so = str(tmp_path_factory.mktemp("recorder") / "libhip_recorder.so")
    subprocess.run(["g++", "-O1", "-std=c++17", "-shared", "-fPIC", "-o", so, os.path.join(HERE, "hip_recorder.cpp")], check=True)
    return so


def record(recorder, jobs, library=None):
    from paper_2505_24196_amd import binding
    res = subprocess.run([sys.executable, os.path.join(HERE, "launch_recorder.py"), recorder, library or binding.LIB_PATH],
                         input=json.dumps(jobs), capture_output=True, text=True, timeout=60)
    assert res.returncode == 0, res.stderr
    return json.loads(res.stdout)


def config(L, d, heads, kv, hd, ffn, vocab, max_seq, max_rows, dtype):
    return [L, d, heads, kv, hd, ffn, vocab, max_seq, max_rows, dtype]


def test_large_lds_is_requested_on_every_device_of_the_process(recorder):
    """A kernel may use more than 64 KiB of LDS only on the devices on which that was asked for: contexts of one process on
    two devices, every family of kernels that goes beyond it."""
    calls = {
        tuple(config(2, 512, 2, 1, 256, 512, 1040, 8192, 32, F32)): [["verify", 32, 8100], ["dp", 8000, 2]],
        tuple(config(2, 4096, 32, 8, 128, 14336, 16400, 2112, 32, BF16)): [["draft", 100], ["verify", 1, 2000], ["verify", 5, 64],
                                                                           ["verify", 8, 2000], ["prefill", 300, 0, 384],
                                                                           ["prefill", 1100, 900, 1152], ["prefill", 2048, 0, 2048]],
        tuple(config(2, 512, 8, 2, 64, 1408, 16400, 2112, 32, BF16)): [["verify", 8, 2000], ["prefill", 1100, 900, 1152]],
    }
    jobs = [{"config": list(c), "device": dev, "calls": k} for dev in (0, 1) for c, k in calls.items()]
    large = {0: set(), 1: set()}
    for done in record(recorder, jobs)["calls"]:
        assert done["rc"] == 0 and done["launches"], done["call"]
        for l in done["launches"]:
            assert l["lds"] <= 160 * 1024
            assert l["lds_allowed"], (done["call"], l)
            if l["lds"] > 64 * 1024:
                large[l["device"]].add(l["kernel"].split("<")[0].split("::")[-1])
    assert large[0] == large[1] == {"gemv_persistent_bf16_kernel", "attn_bf16_kernel", "attn_f32_kernel", "prefill_ring_kernel",
                                    "prefill_attn_lds_kernel"}


def test_prompt_passes_with_the_fp16_form_turned_off(recorder, tmp_path):
    """CLASP_PREFILL_F16_ROWS = 0 (a build-time option: no pass takes fp16 operands): the bf16 form of a pass always leaves the
    sums of its residual projections in the workspace, which has to hold them at every number of rows a pass may have."""
    from paper_2505_24196_amd import build
    so = str(tmp_path / "libclasp_host.so")
    subprocess.run(["hipcc", "--offload-arch=gfx950", "--offload-host-only", "-fuse-cuid=none", "-O1", "-std=c++17", "-shared", "-fPIC",
                    "-Wno-unused-command-line-argument", "-DCLASP_PREFILL_F16_ROWS=0", "-o", so] + build.SOURCES, check=True)
    rows = [(128, 128), (640, 640), (1100, 1152), (4096, 4096), (4097, 4224), (8192, 8192)]
    calls = [["prefill", n, 0, chunk] for n, chunk in rows]
    for done in record(recorder, [{"config": config(2, 4096, 32, 8, 128, 14336, 16400, 8192, 16, BF16), "calls": calls}], so)["calls"]:
        assert done["rc"] == 0, done["call"]
        assert not any("true" in l["kernel"] for l in done["launches"] if "prefill_ring" in l["kernel"])
        for l in done["launches"]:  # kEpiPartial: slices (grid y) of `rows` rows each
            if "prefill_ring_kernel<4," in l["kernel"]:
                assert l["grid"][1] * done["call"][1] <= max(4 * min(done["call"][3], 1024), done["call"][3])


def test_prompt_pass_tests_reach_every_kernel_of_the_prompt_pass(recorder):
    """The GPU test of the prompt passes claims every tile, K-split and attention form: the kernels its shapes and row counts
    launch on 256 CUs are all the ones that are compiled."""
    from tests.test_gpu_kernel_edges import PROMPT_PASSES
    jobs = [{"config": config(3, *shape, 2064, 4224, 32, BF16),
             "calls": [["prefill", n, 0, (n + 127) // 128 * 128] for n in rows]} for shape, rows in PROMPT_PASSES.values()]
    out = record(recorder, jobs)
    assert all(done["rc"] == 0 for done in out["calls"])
    launches = [l for done in out["calls"] for l in done["launches"]]
    compiled = {k for k in out["kernels"] if "clasp::prefill_" in k}
    assert len(compiled) > 40 and compiled == {l["kernel"] for l in launches if "clasp::prefill_" in l["kernel"]}
    splits = {(f16, l["grid"][1]) for l in launches for f16 in ("false", "true") if f"prefill_ring_kernel<4, {f16}," in l["kernel"]}
    assert splits == {(f16, s) for f16 in ("false", "true") for s in (1, 2, 3, 4)}


@pytest.mark.parametrize("V,n,kernels", [
    (16, 7, ["draw_kernel<2>"]), (1024, 7, ["draw_kernel<2>"]),
    (1024, 8, ["chunk_stats_kernel", "draw_kernel<1>"]), (1040, 1, ["chunk_stats_kernel", "draw_kernel<1>"]),
    (4096, 31, ["chunk_stats_kernel", "draw_kernel<1>"]),
    (4112, 1, ["chunk_stats_kernel", "residual_sums_kernel", "draw_kernel<0>"])])
def test_launches_of_an_acceptance_round(recorder, V, n, kernels):
    """One launch for few drafts over few entries, two while a workgroup holds a row in registers, three beyond; the draw of
    clasp_draft_sample takes one launch up to 4096 entries and two beyond."""
    done = record(recorder, [{"config": config(1, 64, 1, 1, 64, 64, V, 32, 32, BF16), "calls": [["accept", n], ["draft", 0]]}])["calls"]
    names = [[l["kernel"].split("(")[0].split("::")[-1] for l in d["launches"]] for d in done]
    assert [d["rc"] for d in done] == [0, 0]
    assert names[0] == kernels
    draw = ["draw_kernel<2>"] if V <= 4096 else ["chunk_stats_kernel", "draw_kernel<0>"]
    assert names[1][-len(draw):] == draw


def test_cache_moves_launch_what_they_move(recorder):
    """bf16 models: four fragments of 1 KiB a workgroup (a block of 32 positions of one head is head_dim / 8 of them), up to 2048
    workgroups; fp32 models: 256 elements, up to 1024."""
    calls = [["kv_load", 1], ["kv_read", 31, 2], ["kv_read", 3, 29], ["kv_load", 4096]]
    done = record(recorder, [{"config": config(1, 512, 8, 2, 64, 64, 112, 4096, 16, dtype), "calls": calls} for dtype in (BF16, F32)])["calls"]
    assert all(d["rc"] == 0 and len(d["launches"]) == 1 for d in done)
    grids = [d["launches"][0]["grid"][0] for d in done]
    assert grids == [2 * 8 // 4, 2 * 2 * 8 // 4, 2 * 8 // 4, 128 * 2 * 8 // 4, 1, 1, 15, 1024]
