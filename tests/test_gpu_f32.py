"""The fp32 model's products (f32.hip) at the edges of their shapes: 1 row, an
odd count, the 16 rows up to which the products take their LayerNorm, and the
first counts past it; one and several chunks of K per wave; two vocabularies
(the heads' last column tile full and ragged).  Logits of each step and the
selection against the oracle on the same history."""
import numpy as np
import pytest

from oracle.decoder import ARDecoder
from paper_2410_13839_amd.workloads import ModelShape, Workload, make_logq, make_prompts, make_weights

from gpu_common import assert_selection_exact, new_session, oracle_logits_at

pytestmark = pytest.mark.gpu

# d, d_ff, vocab, heads K, batch: rows per step = K * batch
CASES = {
    "1 row, d 256": (256, 256, 1025, 1, 1),
    "15 rows, d 512": (512, 768, 65, 5, 3),
    "16 rows, d 2048": (2048, 256, 64, 8, 2),
    "16 rows, d 768": (768, 2048, 33, 2, 8),
    "18 rows (LayerNorm in launches of its own)": (256, 1024, 1025, 3, 6),
    "40 rows, 17 sequences past the heads' LayerNorm": (256, 512, 40, 2, 20),
}


# float32 sums of at most 2048 products of values of order 1: relative error
# below 2048 * 2^-24 = 1.3e-4 of a logit of order 0.5 in the worst case
@pytest.mark.parametrize("name", list(CASES))
def test_f32_decode_rows(name):
    d, f, vocab, K, B = CASES[name]
    shape = ModelShape(n_layers=2, d_model=d, n_heads=d // 64, d_ff=f, k_heads=K, dtype="f32", vocab=vocab,
                       eos_id=vocab - 1, n_phone=40, max_pos=400)
    # three steps; the longest prompts put two 256-key splits and a ragged tail in the attention
    wl = Workload("f32", shape, K=K, top_k=3, batch=B, phon_len=(1, 5), ac_len=(3, 300 if B == 1 else 30),
                  max_new=3 * K, eos_min=3 * K)
    w = make_weights(shape, seed=41)
    logq = make_logq(vocab, eos_id=vocab - 1)
    pr = make_prompts(wl)
    pr.phon = [p % 40 for p in pr.phon]
    pr.ac = [a % (vocab - 1) for a in pr.ac]
    s = new_session(wl, w, logq, topk_max=4)
    s.prefill(pr.phon, pr.ac)
    model = ARDecoder(shape, w)
    emitted = [[] for _ in range(B)]
    for _ in range(3):
        gen = s.seq_state()["gen"].copy()
        tok, cnt = s.step(K, 3)
        lg = s.logits(K)
        for b in range(B):
            ref = oracle_logits_at(model, pr.phon[b], pr.ac[b], emitted[b], K)
            err = float(np.abs(ref - lg[b]).max())
            assert err <= 1e-4, (name, b, err)
            emitted[b].extend(int(x) for x in tok[b][:cnt[b]])
        assert_selection_exact(lg, s.lattice(K, 3), logq, 3, gen, wl.eos_min, shape.eos_id, np.ones(B, bool))
    s.close()
