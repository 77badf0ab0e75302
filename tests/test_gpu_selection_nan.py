"""Selection from logits that hold NaN or infinities (weights or activations
that overflowed): a NaN ranks as -infinity, every chosen id lies in the
vocabulary, and the step and those after it run to their end.  Where every
position has a number to choose from, the lattice is the oracle's on the
logits with -infinity in the NaNs' place, bit for bit."""
import numpy as np
import pytest

from gpu_common import assert_selection_exact, log, new_session
from paper_2410_13839_amd.workloads import ModelShape, Workload, make_logq, make_prompts, make_weights

pytestmark = pytest.mark.gpu

K, TOP_K, V = 4, 4, 1025
SHAPE = ModelShape(n_layers=2, d_model=256, n_heads=4, d_ff=512, k_heads=K, dtype="f32", n_phone=40, max_pos=200)
NUMBERS = [3, 500, 1000]               # ids that keep a number: fewer than top_k


def _bias(kind):
    b = np.zeros((K, V), np.float32)
    if kind == "few numbers":          # every head
        keep = b[:, NUMBERS].copy()
        b[:] = np.nan
        b[:, NUMBERS] = keep
    elif kind == "some NaN":
        b[:, 5:700] = np.nan
    elif kind == "one head all NaN":
        b[2] = np.nan
    elif kind == "all NaN":
        b[:] = np.nan
    else:                              # +inf: emissions are NaN (inf - inf) and -inf
        b[1, [7, 1000]] = np.inf
    return b


@pytest.mark.parametrize("kind", ["few numbers", "some NaN", "one head all NaN", "all NaN", "infinite"])
@pytest.mark.parametrize("mode", ["own", "union", "sample"])
def test_chosen_ids_are_in_the_vocabulary(kind, mode):
    from paper_2410_13839_amd.binding import MTP_LATTICE_OWN, MTP_LATTICE_UNION, MTP_SELECT_SAMPLE
    log(f"{kind}, {mode}: start")
    wl = Workload("nan", SHAPE, K=K, top_k=TOP_K, batch=3, phon_len=(2, 5), ac_len=(5, 20), max_new=6 * K, eos_min=6 * K)
    w = make_weights(SHAPE, seed=3)
    w["b_heads"] = _bias(kind)
    pr = make_prompts(wl)
    pr.phon = [p % 40 for p in pr.phon]
    logq = make_logq()
    s = new_session(wl, w, logq, topk_max=8)
    s.set_selection(MTP_LATTICE_UNION if mode == "union" else MTP_LATTICE_OWN, mode == "union")
    if mode == "sample":
        s.set_sampling(MTP_SELECT_SAMPLE, 1.0, 9)
    s.prefill(pr.phon, pr.ac)
    for _ in range(4):
        gen = s.seq_state()["gen"].copy()
        tok, cnt = s.step(K, TOP_K)
        assert np.all(cnt == K) and np.all((tok >= 0) & (tok < V)), (kind, mode, tok)
        lat = s.lattice(K, TOP_K)
        assert np.all((lat["cand"] >= 0) & (lat["cand"] < V)), (kind, mode)
        if mode == "own" and kind in ("few numbers", "some NaN"):
            lg = s.logits(K)
            lg = np.where(np.isnan(lg), np.float32(-np.inf), lg)
            assert_selection_exact(lg, lat, logq, TOP_K, gen, wl.eos_min, SHAPE.eos_id, np.ones(3, bool))
            if kind == "few numbers":
                assert np.all(np.isin(tok, NUMBERS)), tok
    s.close()
