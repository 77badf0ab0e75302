"""GPU parity of the transition-table estimation (Sec. 3.3: Q derived from
the corpus).  Bigram counts and the input-error tallies must equal the
oracle's exactly; log Q is evaluated in double on both sides and rounded to
float32, so it must agree to within one float32 ulp (the two libraries' double
logarithms may differ in the last bit) with identical -inf entries."""
import numpy as np
import pytest

from gpu_common import log
from oracle.qestimate import bigram_counts, log_q
from paper_2410_13839_amd.workloads import CORPORA, EOS_ID, VOCAB, make_corpus

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


def _gpu(tokens, offsets, V, eos, count_eos, alpha):
    from paper_2410_13839_amd.binding import estimate_logq
    t = torch.from_numpy(np.ascontiguousarray(tokens, np.int32)).cuda()
    o = torch.from_numpy(np.ascontiguousarray(offsets, np.int64)).cuda()
    counts, lq, status = estimate_logq(t, o, V, eos, count_eos, alpha)
    torch.cuda.synchronize()
    return counts.cpu().numpy().view(np.uint32), lq.cpu().numpy(), status.cpu().numpy()


def _ulp_distance(a, b):
    ia = a.view(np.int32).astype(np.int64)
    ib = b.view(np.int32).astype(np.int64)
    ia = np.where(ia < 0, -(ia & 0x7FFFFFFF), ia)
    ib = np.where(ib < 0, -(ib & 0x7FFFFFFF), ib)
    return np.abs(ia - ib)


def _check(tokens, offsets, V, eos, count_eos, alpha):
    C, lq, status = _gpu(tokens, offsets, V, eos, count_eos, alpha)
    rC, bp, bs = bigram_counts(tokens, offsets, V, eos, count_eos)
    assert np.array_equal(C, rC)
    assert status.tolist() == [bp, bs, 0]
    rlq = log_q(rC, alpha)
    inf = np.isneginf(rlq)
    assert np.array_equal(np.isneginf(lq), inf)
    d = _ulp_distance(lq[~inf], rlq[~inf])
    assert d.max(initial=0) <= 1, d.max()
    return C, lq, status


def _ragged(rng, n_seqs, V, max_len, bad):
    lens = rng.integers(0, max_len, size=n_seqs)
    lens[:4] = [0, 1, 2, 0]
    lens[-1] = 50        # skipped when `bad`: frees more tokens than the 3 that utterance 5 then overlaps
    offs = np.concatenate([[0], np.cumsum(lens)]).astype(np.int64)
    toks = rng.integers(0, V, size=int(offs[-1])).astype(np.int32)
    if bad:
        toks[rng.integers(0, len(toks), size=7)] = rng.choice([-1, V, 1 << 20], size=7)
        offs[6] = offs[7] + 3                     # utterance 5 decreasing, 6 also
        offs[-1] = offs[-1] + 5                   # the last one runs past the tokens
    return toks, offs


@pytest.mark.parametrize("count_eos", [False, True])
@pytest.mark.parametrize("bad", [False, True])
@pytest.mark.parametrize("V,alpha", [(33, 0.0), (33, 1.0), (VOCAB, 0.5)])
def test_ragged_corpora_exact(count_eos, bad, V, alpha):
    rng = np.random.default_rng(10 * V + 2 * count_eos + bad)
    toks, offs = _ragged(rng, 700, V - 1, 90, bad)
    _, _, status = _check(toks, offs, V, V - 1, count_eos, alpha)
    if bad:
        assert status[0] > 0 and status[1] >= 2


@pytest.mark.parametrize("case", ["wide_vocab", "long_utterances", "many_utterances"])
def test_every_counting_path(case):
    """The count paths: a vocabulary with more than 64 key buckets (keys
    written one by one), utterance ranges whose spans exceed the LDS bitmap
    (per-utterance walk), and more than a million utterances (offsets read
    from memory)."""
    rng = np.random.default_rng({"wide_vocab": 1, "long_utterances": 2, "many_utterances": 3}[case])
    if case == "wide_vocab":
        V = 2000
        lens = rng.integers(0, 300, size=900)
    elif case == "long_utterances":
        V = VOCAB
        lens = np.array([70000, 3, 0, 90001, 5, 66000])
    else:
        V = 64
        lens = rng.integers(0, 3, size=1_050_000)
    offs = np.concatenate([[0], np.cumsum(lens)]).astype(np.int64)
    toks = rng.integers(0, V - 1, size=int(offs[-1])).astype(np.int32)
    for count_eos in (False, True):
        _check(toks, offs, V, V - 1, count_eos, 1.0)


CHUNK, FROM = 16384, 1 << 23      # positions of a chunk; tokens from which a corpus is counted by chunks


def _cut(rng, total, ends):
    """Ascending offsets over [0, total] that hold `ends` and random ones, a few utterances empty."""
    cuts = np.concatenate([ends, rng.integers(0, total + 1, size=total // 200 + 1)])
    cuts = np.concatenate([cuts, cuts[:3]])
    return np.sort(cuts[(cuts >= 0) & (cuts <= total)]).astype(np.int64)


@pytest.mark.parametrize("total,ends", [
    (1, [0, 1]), (139, [0, 139]), (4097, [3, 4096]),
    (FROM - 1, [0, 3 * CHUNK, FROM - 1]),                     # the last of the general path
    (FROM, [0, CHUNK, FROM]),                                 # an end on a boundary
    (FROM + 1, [7, 2 * CHUNK + 1, FROM]),                     # tokens before the first utterance and past the last
    (FROM + CHUNK - 3, [CHUNK - 1, CHUNK + 1, FROM + CHUNK - 3])])
def test_chunk_edges(total, ends):
    rng = np.random.default_rng(total)
    toks = rng.integers(0, VOCAB - 1, size=total).astype(np.int32)
    if total > 100:
        toks[rng.integers(0, total, size=5)] = VOCAB                  # bad ids are tallied once
    ends = np.array(ends, np.int64)
    for offs in (_cut(rng, total, ends), ends):                       # many utterances; one or two long ones
        if ends[0] > 0:
            offs = offs[offs >= ends[0]]
        for count_eos in (False, True):
            _check(toks, offs, VOCAB, EOS_ID, count_eos, 0.5)


@pytest.mark.parametrize("run", [1, 511, 512, 513, 1024, 5000, 1 << 20])
def test_runs_of_empty_utterances(run):
    """`run` empty utterances at one place: before the first token, inside a chunk, on a chunk's boundary, at the
    end; and a second, shorter run one token on."""
    rng = np.random.default_rng(run)
    toks = rng.integers(0, VOCAB - 1, size=FROM + 5000).astype(np.int32)
    base = _cut(rng, toks.size, np.array([0, toks.size]))
    for at in (0, 3 * CHUNK + 777, 5 * CHUNK, toks.size):
        more = np.concatenate([np.full(run, at), np.full(run // 3, min(at + 1, toks.size))])
        _check(toks, np.sort(np.concatenate([base, more])).astype(np.int64), VOCAB, EOS_ID, True, 0.5)


def test_empty_utterances_cost_little():
    """Eight million empty utterances at the end of a corpus: within eight times the time of the same corpus
    without them (walked one by one they took forty times as long, skipped in doubled steps 1.2 times)."""
    rng = np.random.default_rng(3)
    toks = torch.from_numpy(rng.integers(0, VOCAB - 1, size=FROM + 5000).astype(np.int32)).cuda()
    base = _cut(rng, toks.numel(), np.array([0, toks.numel()]))
    times = []
    for empty in (0, 8 << 20):
        offs = torch.from_numpy(np.concatenate([base, np.full(empty, toks.numel())]).astype(np.int64)).cuda()
        from paper_2410_13839_amd.binding import estimate_logq
        best = float("inf")
        for _ in range(8):
            e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            e0.record()
            estimate_logq(toks, offs, VOCAB, EOS_ID, True, 0.5)
            e1.record()
            torch.cuda.synchronize()
            best = min(best, e0.elapsed_time(e1))
        times.append(best)
    log(f"without and with 8 Mi empty utterances: {times[0] * 1e3:.0f} and {times[1] * 1e3:.0f} us")
    assert times[1] < 8 * times[0]


@pytest.mark.parametrize("V", [1, 2, 181, 182, 1448, 1449])           # 1, 1, 1, 2, 64 and 65 buckets
def test_bucket_edges(V):
    rng = np.random.default_rng(V)
    toks = rng.integers(0, V, size=FROM + 11).astype(np.int32)
    toks[FROM - 30000:] = V - 1                                            # one bucket gets most of a chunk
    offs = _cut(rng, toks.size, np.array([0, 9000, toks.size]))
    _check(toks, offs, V, V - 1, True, 1.0)


def test_descending_offsets_over_many_chunks():
    """The chunk path's result is dropped and its tallies are not added."""
    rng = np.random.default_rng(8)
    toks = rng.integers(0, VOCAB - 1, size=FROM + 100).astype(np.int32)
    toks[[5, 12345, FROM]] = -1
    offs = _cut(rng, toks.size, np.array([0, toks.size]))
    # 40 pairs twice, fewer than the 40,000 utterances without an EOS pair leave out (more pairs
    # than tokens would be refused)
    offs[len(offs) // 2] = offs[len(offs) // 2 - 1] - 40
    offs[-1] += 4
    _check(toks, offs, VOCAB, EOS_ID, False, 0.5)


def test_empty_corpora():
    for toks, offs in ((np.zeros(0, np.int32), np.zeros(1, np.int64)),
                       (np.zeros(0, np.int32), np.zeros(4, np.int64)),
                       (np.array([3], np.int32), np.array([0, 0, 1, 1]))):
        for count_eos in (False, True):
            C, lq, status = _check(toks, offs, 9, 8, count_eos, 1.0)
            assert C.sum() == (1 if (count_eos and len(toks)) else 0)


def test_counts_accumulate_across_calls():
    """Two calls over the two halves of a corpus add up to one call over all of it."""
    from paper_2410_13839_amd.binding import MTP_Q_COUNT_EOS, mtp_q_count, mtp_q_workspace_size
    cp = make_corpus(CORPORA["small"])
    h = len(cp.offsets) // 2
    t = torch.from_numpy(cp.tokens).cuda()
    counts = torch.zeros((VOCAB, VOCAB), dtype=torch.int32, device="cuda")
    status = torch.zeros(3, dtype=torch.int64, device="cuda")
    nb = mtp_q_workspace_size(t.numel(), len(cp.offsets), VOCAB)
    ws = torch.empty(nb, dtype=torch.uint8, device="cuda")
    st = torch.cuda.current_stream()
    for part in (cp.offsets[:h + 1], cp.offsets[h:]):
        o = torch.from_numpy(np.ascontiguousarray(part)).cuda()
        mtp_q_count(t.data_ptr(), t.numel(), o.data_ptr(), o.numel() - 1, VOCAB, EOS_ID, MTP_Q_COUNT_EOS,
                    counts.data_ptr(), status.data_ptr(), ws.data_ptr(), nb, st.cuda_stream)
    torch.cuda.synchronize()
    rC, _, _ = bigram_counts(cp.tokens, cp.offsets, VOCAB, EOS_ID, True)
    assert np.array_equal(counts.cpu().numpy().view(np.uint32), rC)
    assert status.cpu().tolist() == [0, 0, 0]


def test_overlapping_utterances_beyond_the_token_count_are_refused():
    """offsets [0, 8, 0, 8] over 8 tokens: utterances 0 and 2 are the same
    range (16 pairs with the EOS pairs, more than the 8 tokens), utterance 1
    runs backwards.  Nothing is counted; status = [0, 1, 1]."""
    toks = np.arange(8, dtype=np.int32)
    C, lq, status = _gpu(toks, np.array([0, 8, 0, 8], np.int64), 9, 8, True, 1.0)
    assert status.tolist() == [0, 1, 1]
    assert C.sum() == 0
    assert np.all(lq == np.float32(-np.log(9.0)))


def test_libritts_scale_corpus_exact():
    """The 354,780-utterance, ~105 M-token corpus (the benchmark's input):
    every count exact, log Q within one ulp."""
    log("q estimation: generating the corpus")
    cp = make_corpus(CORPORA["libritts_train"])
    log(f"q estimation: {cp.tokens.size} tokens, running")
    C, lq, status = _check(cp.tokens, cp.offsets, VOCAB, EOS_ID, True, 1.0)
    assert status.tolist() == [0, 0, 0]
    assert int(C.sum(dtype=np.int64)) == cp.tokens.size
