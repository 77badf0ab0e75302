"""The products at the edges of their tiles: NAR modules whose row counts take
each row group of the medium kernel, each tile of the four-wave kernel (those of
the residual epilogue at d 1536: 224 rows, and more tiles than workgroups, so
that a workgroup goes on to a second one), each tile height of the eight-wave
kernel (128 .. 256 rows), and their ragged last tiles.
Every row of every utterance is a target, so the stage logits show each output
row; against the float64 oracle within the bf16 tolerance of test_gpu_nar.py
(two layers: 3e-2 is twice what twelve show)."""
import numpy as np
import pytest

from gpu_common import log
from oracle.nar import NARModel
from paper_2410_13839_amd.workloads import ModelShape, NarWorkload, make_nar_inputs, make_weights

pytestmark = pytest.mark.gpu

# rows -> the row groups or tiles of the products of 3072 (QKV), 4096 (FFN1) and
# 1024 columns (split K, or with the residual), d 1024 over 256 CUs
ROWS = {
    1: "medium kernel, 16-row groups",
    17: "medium, 16 rows (one in the last group), four splits",
    33: "medium, 32 rows",
    65: "medium, 64 rows",
    192: "medium, 64 rows, the last full group",
    193: "64 x 64 (one row in the last tile), 64 x 64, medium unsplit / in two splits",
    257: "64 x 64, 64 x 64, medium unsplit / 64 x 64 split (one row in the last tile)",
    768: "64 x 64 in QKV and FFN1, the most workgroups of three per CU",
    1025: "128 x 64 (one row in the last tile), 128 x 64, 64 x 64 in two splits / 128 x 64 split",
    1536: "128 x 64, 128 (eight waves), 64 x 64 / 128 x 64",
    2049: "128, 160 (one row in the last tile), 64 x 64 / 128 x 64",
    2720: "160, 192, 64 x 64 / 128 x 64",
    4001: "192, 256, 128 with the residual",
    4090: "224, 256, 128",
    8209: "224, 192, 160",
    10250: "256, 224, 192",
}


@pytest.mark.parametrize("rows", list(ROWS))
def test_every_row_of_a_tiled_product(rows):
    _check(rows, 1024)


# d 512: QKV has 1536 columns, FFN1 2048; the last and the first rows past one round of the medium kernel
@pytest.mark.parametrize("rows", [256, 257, 320, 321, 1024, 1025])
def test_narrow_products_at_one_round_of_the_medium_kernel(rows):
    _check(rows, 512)


# d 1536, 512 workgroups: the residual epilogue's tiles of 128 columns
WIDE = {8065: "224 rows (one in the last tile), three stages", 9409: "128 rows, 888 tiles",
        13000: "160 rows, 984 tiles"}


@pytest.mark.parametrize("rows", list(WIDE))
def test_residual_tiles_of_the_wide_model(rows):
    """The first and last two utterances and every eighth."""
    _check(rows, 1536, 256, lambda b, n: b < 2 or b >= n - 2 or b % 8 == 0)


# d 2048, FFN2 with K = 8192: the last row count of 64 x 64 tiles, the first of 128 x 64 (one row in the last)
@pytest.mark.parametrize("rows", [384, 385])
def test_split_products_of_the_longest_k(rows):
    _check(rows, 2048)


def _check(rows, d, d_ff=None, which=lambda b, n: True):
    shape = ModelShape(n_layers=2, d_model=d, n_heads=d // 64, d_ff=d_ff or 4 * d, k_heads=1, dtype="bf16", vocab=257, eos_id=256,
                       n_phone=8, max_pos=160, nar=True)
    # utterances of 97 rows (odd starts in the tiles) and a rest
    n, rest = divmod(rows, 97)
    lens = [97] * n + ([rest] if rest else [])
    wl = NarWorkload("tiles", shape, batch=len(lens), phon_len=(0, 0), prompt_len=(0, 0), target_len=(1, 97))
    w = make_weights(shape, seed=43)
    inp = make_nar_inputs(wl, seed_base=900)
    rng = np.random.default_rng(rows)
    inp.a1 = [rng.integers(0, shape.codebook, size=t).astype(np.int32) for t in lens]
    from paper_2410_13839_amd.binding import NarSession
    s = NarSession(shape, w, max_batch=len(lens), max_seq=97)
    s.prepare(inp.phon, inp.prompt, inp.a1)
    s.run()
    got = s.logits(0)
    s.close()
    m = NARModel(shape, w)
    worst, o = 0.0, 0
    for b, t in enumerate(lens):
        if not which(b, len(lens)):
            o += t
            continue
        h = m.forward(m.embed(2, inp.phon[b], inp.prompt[b], inp.a1[b][None]))
        err = float(np.max(np.abs(got[o:o + t] - m.stage_logits(h, 2))))
        worst = max(worst, err)
        assert err < 3e-2, (rows, b, err)
        o += t
    log(f"{rows} rows: max |logit err| {worst:.3g}")
