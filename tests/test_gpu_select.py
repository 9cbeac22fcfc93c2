"""GPU parity of cc_select against the oracle: bit-exact scores, indices, count."""
import numpy as np
import pytest
import torch

import paper_2510_10129_amd as cc
from paper_2510_10129_amd import _lib
from oracle import select as osel
from workloads import CONFIGS, gen

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.fixture(scope="module")
def ctx():
    c = cc.Context(d=256, H_q=4, H_kv=2, d_h=64, f=1024, rope_base=1e4, rms_eps=1e-5,
                   N_cap=1024, M_cap=64, T_cap=131072)
    yield c
    c.close()


def _run(ctx, A, bp, w, tau=0, flags=0, off=0, tail=0):
    At = torch.from_numpy(A).to(DEV)
    idx, n = ctx.select(At, bp, w, tau, flags, off, tail)
    return idx[:n].cpu().numpy(), n


def _check(ctx, A, bp, w, tau=0, grouping=True, off=0, tail=0):
    got, n = _run(ctx, A, bp, w, tau, 0 if grouping else _lib.FLAG_NO_GROUPING, off, tail)
    ref = osel.select(A, bp, w, tau, grouping, off, tail)
    assert n == len(ref)
    assert np.array_equal(got, ref)
    return n


def test_scores_bit_exact(ctx):
    rng = np.random.default_rng(0)
    for Qa, T in ((1, 1), (3, 65), (32, 1024), (100, 777), (128, 16384)):
        A = rng.random((Qa, T), dtype=np.float32)
        At = torch.from_numpy(A).to(DEV)
        s = torch.empty(T, dtype=torch.float32, device=DEV)
        ctx.step_column_scores(At, s)
        assert np.array_equal(s.cpu().numpy().view(np.uint32), osel.column_scores(A).view(np.uint32))


@pytest.mark.parametrize("name", ["C1", "C2", "C3", "C4", "C5"])
def test_configs_bit_exact(ctx, name):
    wl = CONFIGS[name]
    A = gen.aux_attention(wl)
    for bp in wl.recomp_bp:
        n = _check(ctx, A, bp, wl.window, wl.tau, True, wl.P, wl.Q)
        print(f"{name} recomp {bp / 100:.0f}%: k={wl.T * bp // 10000} -> M={n} (M_sel/T={(n - wl.Q) / wl.T:.3f})")
    _check(ctx, A, wl.recomp_bp[0], wl.window, wl.tau, False, wl.P, wl.Q)


def test_random_ragged_with_heavy_ties(ctx):
    rng = np.random.default_rng(1)
    for it in range(40):
        T = int(rng.integers(1, 6000))
        Qa = int(rng.integers(1, 9))
        w = int(rng.integers(1, 70))
        tau = int(rng.integers(0, w + 1))
        bp = int(rng.choice([0, 1, 500, 2000, 5000, 9999, 10000]))
        A = rng.integers(0, 4, size=(Qa, T)).astype(np.float32) * 0.25     # few distinct sums
        _check(ctx, A, bp, w, tau, bool(it % 3), int(rng.integers(0, 100)), int(rng.integers(0, 40)))


def test_degenerate_cases(ctx):
    A = np.full((4, 300), 0.125, dtype=np.float32)           # all equal: lowest indices win
    got, n = _run(ctx, A, 2000, 8, 5, off=10, tail=3)
    # k = 60 candidates 0..59; the last passing window starts at 55 (55..59 = 5 candidates) and ends at 62
    assert got.tolist() == list(range(10, 73)) + [310, 311, 312]
    assert np.array_equal(got, osel.select(A, 2000, 8, 5, True, 10, 3))
    _check(ctx, A, 0, 8, 5, True, 0, 0)                      # nothing at all
    _check(ctx, A, 10000, 8, 5, True, 0, 0)                  # everything
    _check(ctx, np.zeros((2, 50), np.float32), 5000, 8)      # zeros incl. default tau
    neg = np.zeros((1, 64), np.float32); neg[0, ::2] = -0.0
    _check(ctx, neg, 2500, 4, 2)                             # -0 == +0
    wide = np.random.default_rng(3).random((2, 5000)).astype(np.float32)
    _check(ctx, wide, 3000, 1024, 300)                       # widest window
    _check(ctx, wide[:, :7], 5000, 32, 2)                    # window longer than T
    big = np.random.default_rng(4).random((2, 131072)).astype(np.float32)
    _check(ctx, big, 2000, 16)                               # T at capacity


def test_long_inputs_with_ties_and_crowded_threshold_digit(ctx):
    """Paths of the selection kernel that short inputs do not reach: more keys share the
    threshold's leading digit than its LDS list holds (the remaining digits then come from further
    passes over the scores), with and without equal scores at the threshold."""
    rng = np.random.default_rng(6)
    T = 100000
    few = rng.integers(1, 5, size=(3, T)).astype(np.float32) * 0.125           # ten distinct sums: crowded, tied
    _check(ctx, few, 2000, 16, 0, True, 7, 3)
    _check(ctx, few, 5000, 8, 5, False, 0, 0)
    narrow = (1.0 + rng.random((1, T)) * 0.1).astype(np.float32)                 # one binade, all distinct (mostly)
    _check(ctx, narrow, 2000, 16, 0, True, 0, 0)
    mixed = narrow.copy()
    mixed[0, ::3] = np.float32(1.05)                                            # a third of the keys equal, threshold among them
    _check(ctx, mixed, 5000, 32, 0, True, 64, 128)


def test_strided_input_and_async_count(ctx):
    rng = np.random.default_rng(5)
    full = torch.from_numpy(rng.random((16, 1000), dtype=np.float32)).to(DEV)
    view = full[:, 100:740]                                  # ld = 1000, T = 640
    idx, n = ctx.select(view, 2000, 8, 5, 0, 0, 0)
    ref = osel.select(view.cpu().numpy(), 2000, 8, 5)
    assert n == len(ref) and np.array_equal(idx[:n].cpu().numpy(), ref)
    n_out = torch.zeros(1, dtype=torch.int32, device=DEV)
    idx2, none = ctx.select(view, 2000, 8, 5, n_out=n_out, sync=False)
    torch.cuda.synchronize()
    assert none is None and int(n_out.item()) == n and torch.equal(idx2[:n], idx[:n])


def test_argument_errors(ctx):
    A = torch.zeros((2, 64), dtype=torch.float32, device=DEV)
    for kw, code in ((dict(recomp_bp=10001, window=8), _lib.CC_ERR_SHAPE),
                     (dict(recomp_bp=100, window=0), _lib.CC_ERR_SHAPE),
                     (dict(recomp_bp=100, window=2000), _lib.CC_ERR_SHAPE),
                     (dict(recomp_bp=100, window=8, tau=9), _lib.CC_ERR_SHAPE),
                     (dict(recomp_bp=100, window=8, n_tail=-1), _lib.CC_ERR_SHAPE)):
        with pytest.raises(cc.CacheClipError) as e:
            ctx.select(A, **kw)
        assert e.value.status == code
    small = cc.Context(d=256, H_q=4, H_kv=2, d_h=64, f=1024, rope_base=1e4, rms_eps=1e-5,
                       N_cap=64, M_cap=8, T_cap=32)
    with pytest.raises(cc.CacheClipError) as e:
        small.select(A, 100, 8)
    assert e.value.status == _lib.CC_ERR_WORKSPACE
    small.close()


# ------------------------------------------------- scores from batched per-chunk attention
def _dev_blocks(blocks_np, pad_rows=0, pad_cols=0):
    """Device copies; with padding the blocks become strided views of larger tensors."""
    out = []
    for A, c0, L in blocks_np:
        H, Qa, W = A.shape
        big = torch.full((H, Qa + pad_rows, W + pad_cols), 123.0, dtype=torch.float32, device=DEV)
        big[:, :Qa, :W] = torch.from_numpy(A).to(DEV)
        out.append((big[:, :Qa, :W], c0, L))
    return out


@pytest.mark.parametrize("H,Qa,P,lens", [
    (1, 1, 0, [1]),
    (3, 5, 4, [63, 64, 65, 1, 200]),
    (14, 33, 16, [300, 17, 511]),
    (16, 128, 64, [1024, 777]),
    (28, 70, 8, [129] * 5),
    (9, 64, 0, [40] * 70),            # more batch elements than one launch takes
])
def test_block_scores_bit_exact(ctx, H, Qa, P, lens):
    rng = np.random.default_rng(H * 1000 + Qa)
    blocks = [(rng.random((H, Qa, P + L + Qa), dtype=np.float32), P, L) for L in lens]
    ref = osel.block_scores(blocks)
    for pad in (0, 3):
        score = torch.full((sum(lens),), -1.0, dtype=torch.float32, device=DEV)
        ctx.step_block_scores(_dev_blocks(blocks, pad, pad), score)
        torch.cuda.synchronize()
        assert np.array_equal(score.cpu().numpy().view(np.uint32), ref.view(np.uint32)), (H, Qa, pad)


def test_select_blocks_matches_oracle(ctx):
    rng = np.random.default_rng(11)
    for H, Qa, P, lens, bp, w in ((4, 16, 8, [256] * 4, 2000, 8), (14, 32, 16, [300, 100, 511, 77], 1000, 16),
                                  (2, 3, 0, [50], 5000, 4)):
        # peaked rows: a few columns carry most of the weight, with ties across heads
        blocks = []
        for L in lens:
            A = rng.random((H, Qa, P + L + Qa), dtype=np.float32) * 0.01
            hot = rng.integers(P, P + L, size=max(1, L // 10))
            A[:, :, hot] += rng.integers(1, 4, size=(1, 1, len(hot))).astype(np.float32) * 0.25
            blocks.append((A, P, L))
        s = osel.block_scores(blocks)
        for grouping in (True, False):
            ref = osel.select_from_scores(s, bp, w, 0, grouping, P, Qa)
            idx, n = ctx.select_blocks(_dev_blocks(blocks), bp, w, 0, 0 if grouping else _lib.FLAG_NO_GROUPING, P, Qa)
            assert n == len(ref) and np.array_equal(idx[:n].cpu().numpy(), ref)


def test_block_scores_argument_errors(ctx):
    A = torch.zeros((2, 4, 40), dtype=torch.float32, device=DEV)
    score = torch.zeros(64, dtype=torch.float32, device=DEV)
    with pytest.raises(ValueError):
        ctx.step_block_scores([(A, 30, 20)], score)                     # block runs past its width
    with pytest.raises(ValueError):
        ctx.step_block_scores([(A, 0, 10), (A[:1], 0, 10)], score)      # differing head counts
    arr = (_lib._AuxBlock * 1)(_lib._AuxBlock(A.data_ptr(), A.stride(0), A.stride(1), 0, 0))
    assert ctx._lib.cc_step_block_scores(ctx._h, arr, 1, 2, 4, score.data_ptr()) == _lib.CC_ERR_SHAPE   # len 0
    arr = (_lib._AuxBlock * 1)(_lib._AuxBlock(A.data_ptr(), A.stride(0), 10, 0, 20))
    assert ctx._lib.cc_step_block_scores(ctx._h, arr, 1, 2, 4, score.data_ptr()) == _lib.CC_ERR_SHAPE   # rows overlap
    arr = (_lib._AuxBlock * 1)(_lib._AuxBlock(None, A.stride(0), A.stride(1), 0, 20))
    assert ctx._lib.cc_step_block_scores(ctx._h, arr, 1, 2, 4, score.data_ptr()) == _lib.CC_ERR_NULL
    small = cc.Context(d=256, H_q=4, H_kv=2, d_h=64, f=1024, rope_base=1e4, rms_eps=1e-5,
                       N_cap=64, M_cap=8, T_cap=32)
    with pytest.raises(cc.CacheClipError) as e:
        small.select_blocks([(A, 0, 40)], 1000, 8)
    assert e.value.status == _lib.CC_ERR_WORKSPACE
    small.close()


@pytest.mark.parametrize("name,prefix", [("C2", None), ("C2", 0), ("C4", None)])
def test_blocks_window_sweep_and_no_prefix(ctx, name, prefix):
    """Per-chunk-normalised scores from batched tensors at request size: windows 8, 16, 32,
    grouping on and off, with and without a shared prefix, ragged chunk lengths (C4)."""
    import dataclasses
    wl = CONFIGS[name]
    if name == "C4":       # a third of the request keeps the host-side generator quick
        wl = dataclasses.replace(wl, chunk_lens=wl.chunk_lens[:10], Q_a=32)
    blocks = gen.aux_attention_blocks(wl, heads=14 if name == "C2" else 9, prefix=prefix)
    P = blocks[0][1]
    s = osel.block_scores(blocks)
    assert abs(float(s.sum()) - wl.Q_a * len(blocks)) < 0.5 * wl.Q_a * len(blocks)   # most mass sits on chunk tokens
    dev_blocks = _dev_blocks(blocks)
    score = torch.empty(wl.T, dtype=torch.float32, device=DEV)
    ctx.step_block_scores(dev_blocks, score)
    assert np.array_equal(score.cpu().numpy().view(np.uint32), s.view(np.uint32))
    for w in (8, 16, 32):
        for grouping in (True, False):
            ref = osel.select_from_scores(s, 2000, w, 0, grouping, P, wl.Q)
            idx, n = ctx.select_blocks(dev_blocks, 2000, w, 0, 0 if grouping else _lib.FLAG_NO_GROUPING, P, wl.Q)
            assert n == len(ref) and np.array_equal(idx[:n].cpu().numpy(), ref), (name, prefix, w, grouping)
        print(f"{name} prefix={P} w={w}: M_sel/T = {(len(osel.select_from_scores(s, 2000, w, 0, True, P, wl.Q)) - wl.Q) / wl.T:.3f}")


@pytest.mark.parametrize("T", [16384, 16385, 20479, 20480, 20481, 20545, 24575, 24576, 45001, 131072])
def test_selection_by_several_workgroups_edges(ctx, T):
    """Both sides of the size where several workgroups share a selection and of its 4096-token
    tiles: windows that reach over tile edges (up to 1024 tokens), equal scores at the threshold in
    many tiles, one score alone, a threshold bin over and under its list, every token and none."""
    rng = np.random.default_rng(T)
    smooth = rng.random((2, T)).astype(np.float32)
    runs = smooth.copy()
    for e in range(4096, T, 4096):                        # runs of high scores across tile edges
        runs[:, e - 300:e + 300] += 2.0
    runs[:, -40:] += 2.0                                  # and at the end
    for w, tau in ((1, 0), (7, 0), (64, 20), (65, 0), (1000, 400), (1024, 1)):
        _check(ctx, runs, 2000, w, tau, True, 5, 3)
    _check(ctx, smooth, 2000, 16, 0, False, 0, 0)
    tied = rng.integers(1, 6, size=(1, T)).astype(np.float32) * 0.25        # crowded: five values, one bin each
    _check(ctx, tied, 3000, 16, 0, True, 1, 2)
    some = smooth.copy()
    some[:, rng.choice(T, size=min(T // 2, 7000), replace=False)] = 0.5    # equal sums at the median, within the list
    for bp in (4500, 5000, 6000):
        _check(ctx, some, bp, 8, 0, True, 0, 1)
    spread = np.exp(rng.standard_normal((1, T)) * 12.0).astype(np.float32)  # many binades, zeros and one huge score
    spread[0, ::3] = 0.0
    spread[0, T // 2] = 3e38
    for bp in (1, 1500, 6600, 6700, 9999):
        _check(ctx, spread, bp, 16, 1, True, 64, 0)
    _check(ctx, np.full((1, T), 0.125, np.float32), 5000, 8, 5, True, 0, 0)
    for bp in (0, 10000):
        _check(ctx, smooth, bp, 8, 0, True, 2, 7)


def test_block_scores_leave_ranges_for_the_selection(ctx):
    """Several score launches (more batch elements than one takes, ragged, shorter than a workgroup's
    columns) in front of a selection by one workgroup and by several."""
    rng = np.random.default_rng(3)
    for lens in ([40] * 70, [1] * 130, [int(v) for v in rng.integers(1, 600, size=80)]):
        blocks = [(rng.random((2, 3, 2 + L + 3), dtype=np.float32), 2, L) for L in lens]
        ref = osel.select_from_scores(osel.block_scores(blocks), 3000, 8, 0, True, 2, 3)
        idx, n = ctx.select_blocks(_dev_blocks(blocks), 3000, 8, 0, 0, 2, 3)
        assert n == len(ref) and np.array_equal(idx[:n].cpu().numpy(), ref), len(lens)


def _order_by_key(score):
    """Candidates' order by the key of the score's bits (larger first, then the lower token): the order of
    the numbers where they are numbers, infinities and NaN (above them, by its bits) included."""
    u = (score + np.float32(0.0)).view(np.uint32)
    key = np.where(u >> 31, ~u, u | np.uint32(0x80000000)).astype(np.int64)
    return np.lexsort((np.arange(len(key)), -key))


def _check_by_key(ctx, A, bp, w, off=0, tail=0):
    s = osel.column_scores(A)
    T = len(s)
    cand = np.zeros(T, bool)
    cand[_order_by_key(s)[:osel.candidate_count(T, bp)]] = True
    ref = np.r_[off + np.nonzero(osel.group_windows(cand, w, osel.default_tau(w)))[0], off + T + np.arange(tail)]
    got, n = _run(ctx, A, bp, w, 0, 0, off, tail)
    assert n == len(ref) and np.array_equal(got, ref), (T, bp, w)


def _crowded(kind, T, rng):
    if kind == "zero":                  # scores within an octave and one that stretches the range of the keys
        s = (1.0 + 0.9 * rng.random((1, T))).astype(np.float32)
        s[0, T // 3] = 0.0
    elif kind == "equal":
        s = np.full((1, T), 0.125, np.float32)
    elif kind == "steps":               # a handful of values: the threshold's ties run over many tiles
        s = rng.integers(1, 6, size=(1, T)).astype(np.float32) * 0.25
    elif kind == "low bits":            # two values that differ in the last bit, and a zero far below
        s = np.where(rng.random((1, T)) < 0.5, np.float32(0.7), np.nextafter(np.float32(0.7), np.float32(1))).astype(np.float32)
        s[0, 5] = 0.0
    else:                               # "few below": nearly all keys above the threshold's bin, most of it tied
        s = np.full((1, T), 3.0, np.float32)
        s[0, rng.choice(T, T // 2, replace=False)] = 1.0
        s[0, rng.choice(T, 9, replace=False)] = 1e-30
    return s


@pytest.mark.parametrize("kind", ["zero", "equal", "steps", "low bits", "few below"])
@pytest.mark.parametrize("T", [20545, 24576, 65539, 131072])
def test_threshold_bin_with_more_keys_than_the_list(ctx, T, kind):
    """Several workgroups with most of the scores in the threshold's bin: digits and ties from all
    scores, at sizes that end a tile, a 16-byte load and a word, at ratios whose threshold lies in different tiles."""
    rng = np.random.default_rng(T)
    s = _crowded(kind, T, rng)
    for bp, w in ((1, 1), (2000, 16), (5000, 32), (7777, 8), (9999, 64), (3000, 1000)):
        _check_by_key(ctx, s, bp, w, 3, 5)


@pytest.mark.filterwarnings("ignore:overflow encountered")
@pytest.mark.parametrize("T", [16384, 24576, 40001])
def test_infinite_and_nan_scores(ctx, T):
    """Sums that overflow to infinity, and NaN, take part by the order of their bits in every path."""
    rng = np.random.default_rng(T)
    s = rng.random((2, T)).astype(np.float32)
    s[:, rng.choice(T, 300, replace=False)] = 3e38                   # their sum is infinite
    for bp in (50, 1000, 6000):
        _check_by_key(ctx, s, bp, 16)
    s[0, rng.choice(T, 200, replace=False)] = np.nan
    for bp in (50, 1000, 6000):
        _check_by_key(ctx, s, bp, 16, 1, 2)
    _check_by_key(ctx, np.full((2, T), 3e38, np.float32), 3000, 8)   # nothing but infinities


def test_crowded_selection_is_shared_by_the_workgroups(ctx):
    """A crowded threshold bin costs a few passes over the scores (measured: see select.hip), not a selection by
    one workgroup after the others, which took four times the ordinary call."""
    T, idx = 65536, torch.empty(65536 + 8, dtype=torch.int32, device=DEV)
    n = torch.empty(1, dtype=torch.int32, device=DEV)
    rng = np.random.default_rng(0)
    us = {}
    for kind in ("ordinary", "zero", "equal", "steps"):
        s = np.exp(rng.standard_normal((1, T))).astype(np.float32) if kind == "ordinary" else _crowded(kind, T, rng)
        At, best = torch.from_numpy(s).to(DEV), 1e9
        for _ in range(5):
            ctx.profile_enable(True)
            ctx.profile_read()
            for _ in range(10):
                ctx.select(At, 2000, 16, 0, 0, 0, 8, idx, n, sync=False)
            ms, count = ctx.profile_read()["select"]
            ctx.profile_enable(False)
            best = min(best, ms * 1e3 / count)
        us[kind] = best
    print({k: round(v, 1) for k, v in us.items()})
    assert max(us.values()) < 3 * us["ordinary"], us


def _ties_across_the_cut(T, k, n, rng):
    """Scores that all differ but for n in a row by rank, of which the first k take about half."""
    lo = min(max(k - n // 2, 0), max(T - n, 0))
    by_rank = (1.0 - np.arange(T) / (2.0 * T)).astype(np.float32)
    by_rank[lo:lo + n] = by_rank[lo]
    a = np.empty((1, T), np.float32)
    a[0, rng.permutation(T)] = by_rank
    assert T <= n or not 0 < k < T or (lo < k < lo + n and (a == by_rank[lo]).sum() == n)
    return a


@pytest.mark.parametrize("window", [1, 16, 64, 65])
@pytest.mark.parametrize("T", [1, 17, 64, 4095, 4097, 8192, 20480])
def test_one_workgroup_selection_edges(ctx, T, window):
    """Rows of 4096 keys that end anywhere, thresholds inside 64 and 65 equal scores (the most that are ranked in a
    list, and one more) and inside all of them, scores whose range makes the first bins one key wide or crowds them, no
    and all tokens; the count on the device is the one handed back."""
    rng = np.random.default_rng(T + window)
    spread = rng.random((1, T), dtype=np.float32)
    far = 1.0 + spread
    far[0, T // 2] = 0.0
    cases = [(a, bp) for a in (spread, np.full((1, T), 0.25, np.float32), (1.0 + spread * 2.0 ** -13).astype(np.float32), far)
             for bp in (0, 700, 2500, 10000)]
    cases += [(_ties_across_the_cut(T, T * bp // 10000, n, rng), bp) for n in (64, 65) for bp in (700, 2500)]
    for a, bp in cases:
        At = torch.from_numpy(a).to(DEV)
        n_dev = torch.full((1,), -1, dtype=torch.int32, device=DEV)
        idx, n = ctx.select(At, bp, window, 0, 0, 5, 3, n_out=n_dev)
        ref = osel.select(a, bp, window, 0, True, 5, 3)
        assert n == len(ref) == int(n_dev.item())
        assert np.array_equal(idx[:n].cpu().numpy(), ref)
