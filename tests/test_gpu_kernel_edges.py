"""Kernels at the sizes where their tilings and dispatch rules end: remainders of a K split, one workgroup too few or too
many, the smallest and largest of a range. Everything goes through the C ABI and is compared with the CPU oracle or a
plain PyTorch float64 evaluation of the same formula."""
import numpy as np
import pytest
import torch

import synth_inputs as si
from oracle import clasp_oracle as oc
from tests.test_gpu_parity import assert_close

pytestmark = pytest.mark.gpu


def build(shape, max_seq, max_rows=32, seed=3):
    import paper_2505_24196_amd as clasp
    model = si.gen_model(shape, seed, "cpu")
    return clasp.Engine(shape, max_seq=max_seq, max_rows=max_rows).load(model), oc.OracleModel(shape, si.model_to_numpy(model))


def verify_against_oracle(shape, row_counts, tol, max_seq=128):
    """Verify passes of the given row counts chained on one cache: all states and logits of every row."""
    eng, om = build(shape, max_seq)
    cache = oc.KVCache(shape, max_seq)
    toks = [int(t) for t in si.gen_tokens(5, sum(row_counts), shape.vocab)]
    pos = 0
    for n in row_counts:
        out = eng.clasp_verify_forward(torch.tensor(toks[pos:pos + n], dtype=torch.int32, device="cuda"), pos,
                                       want_hidden=True, want_logits=True)
        ref = [om.token(t, pos + i, cache, want_states=True) for i, t in enumerate(toks[pos:pos + n])]
        assert_close(out["hidden"].cpu().numpy(), np.stack([r[0] for r in ref], 1), tol, f"{n} rows at {pos}: hidden")
        assert_close(out["logits"].cpu().numpy(), np.stack([r[1] for r in ref]), tol, f"{n} rows at {pos}: logits")
        pos += n
    eng.close()


# The fp32 projections split K/16 steps over eight wavefronts and take them four at a time: K = 48 leaves wavefronts
# without a step, 80 and 272 give unequal slices, 2064 gives several rounds of both stage sets with a remainder. Error of
# one sum of K products: about sqrt(K) * 2^-24 of its size, 2.7e-6 at 2064; four of them per layer, two layers.
@pytest.mark.parametrize("d,heads,kv,hd,ffn", [(48, 3, 1, 16, 80), (272, 17, 17, 16, 48), (256, 4, 2, 64, 2064)])
def test_fp32_projections_with_uneven_k_slices(d, heads, kv, hd, ffn):
    shape = si.ModelShape("edge-f32", 2, d, heads, kv, hd, ffn, 112, "f32")
    verify_against_oracle(shape, (1, 5, 16, 17, 32), 2e-5)
