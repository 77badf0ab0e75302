"""Prefill attention at the edges of its tiles: sequences around the 64-row
tile and the 64-key block, few of them (two wave groups share the keys) and
many (one group), head counts with and without the per-XCD numbering, causal
(decoder) and bidirectional (NAR).  The query and key weights are scaled so
that scores spread over some 20 nats and a row's softmax reference moves from
block to block.

Against the oracle with the same bfloat16 roundings (what is left is the order
of the sums and the probabilities' rounding): 3e-2 as for the bf16 models in
test_gpu_nar.py; a block weighed by a wrong reference is off by more than 0.1."""
import numpy as np
import pytest

from gpu_common import log, oracle_logits_at
from oracle.decoder import ARDecoder
from oracle.nar import NARModel
from paper_2410_13839_amd.workloads import (ModelShape, NarWorkload, bf16_round, make_logq, make_nar_inputs,
                                            make_weights)

pytestmark = pytest.mark.gpu

LENS = [1, 15, 63, 64, 65, 127, 128, 129, 192, 193, 257, 300]


def _weights(shape):
    w = make_weights(shape, seed=91)
    d = shape.d_model
    for i in range(shape.n_layers):
        a = w[f"l{i}.w_qkv"].copy()
        a[:2 * d] *= 4.0 * np.sqrt(512 / d)
        w[f"l{i}.w_qkv"] = bf16_round(a.astype(np.float32))
    return w


# (d_model, heads, copies of every length): tiles x heads <= 512 takes two groups
@pytest.mark.parametrize("d,heads,copies", [(512, 8, 1), (256, 4, 1), (512, 8, 3), (256, 4, 6)])
def test_bidirectional(d, heads, copies):
    shape = ModelShape(n_layers=1, d_model=d, n_heads=heads, d_ff=256, k_heads=1, dtype="bf16", vocab=129, eos_id=128,
                       n_phone=8, max_pos=320, nar=True)
    lens = LENS * copies
    wl = NarWorkload("attn", shape, batch=len(lens), phon_len=(0, 0), prompt_len=(0, 0), target_len=(1, 300))
    w = _weights(shape)
    inp = make_nar_inputs(wl, seed_base=77)
    rng = np.random.default_rng(5)
    inp.a1 = [rng.integers(0, shape.codebook, size=t).astype(np.int32) for t in lens]
    from paper_2410_13839_amd.binding import NarSession
    s = NarSession(shape, w, max_batch=len(lens), max_seq=300)
    s.prepare(inp.phon, inp.prompt, inp.a1)
    s.run()
    got = s.logits(0)
    s.close()
    m = NARModel(shape, w, emulate_bf16=True)
    worst, o = 0.0, 0
    for b, t in enumerate(lens):
        if b < len(LENS) or b >= len(lens) - 2:
            ref = m.stage_logits(m.forward(m.embed(2, inp.phon[b], inp.prompt[b], inp.a1[b][None])), 2)
            err = float(np.max(np.abs(got[o:o + t] - ref)))
            worst = max(worst, err)
            assert err < 3e-2, (b, t, err)
        o += t
    log(f"d {d}, {heads} heads, {len(lens)} sequences: max |logit err| {worst:.3g}")


@pytest.mark.parametrize("copies", [1, 3])
def test_causal(copies):
    """Two layers, so the last row's logits depend on every row."""
    shape = ModelShape(n_layers=2, d_model=512, n_heads=8, d_ff=256, k_heads=1, dtype="bf16", n_phone=8, max_pos=320)
    lens = LENS * copies
    w = _weights(shape)
    rng = np.random.default_rng(6)
    ac = [rng.integers(0, 1024, size=t).astype(np.int32) for t in lens]
    phon = [np.zeros(0, np.int32)] * len(lens)
    from paper_2410_13839_amd.binding import Session
    s = Session(shape, w, make_logq(), max_batch=len(lens), max_prompt=300, max_new=4, eos_min=4, topk_max=8)
    s.prefill(phon, ac)
    s.step(1, 1)
    got = s.logits(1)
    s.close()
    m = ARDecoder(shape, w, emulate_bf16=True)
    worst = 0.0
    for b, t in enumerate(lens):
        if b < len(LENS) or b >= len(lens) - 2:
            err = float(np.max(np.abs(got[b] - oracle_logits_at(m, phon[b], ac[b], [], 1))))
            worst = max(worst, err)
            assert err < 3e-2, (b, t, err)
    log(f"causal, {len(lens)} sequences: max |logit err| {worst:.3g}")
