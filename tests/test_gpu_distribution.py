"""The selection kernels at the edges of their dispatch: the scores-in filter's
block widths and step lengths, rows gathered and ordered by distribution (and
the rows that leave that way for the general sort), radix selection over a
row's own span, and the union's bitmap and its span limit. Everything is
compared bit for bit with the oracle: the selections compute no score."""
import numpy as np
import pytest
import torch

from oracle import litetopk_oracle as orc
from paper_2607_11976_amd import litetopk as lt
from paper_2607_11976_amd import workloads
from parity import check_row_exact
from helpers import oracle_topk, to_dev

pytestmark = pytest.mark.gpu


def _rows(kind, nq, nk, seed):
    rng = np.random.default_rng(seed)
    if kind in ("normal", "ties", "special", "const"):
        return workloads.score_rows(nq, nk, seed=seed, kind=kind, ld=(nk + 3) // 4 * 4)
    s = np.empty((nq, (nk + 3) // 4 * 4), dtype=np.float32)
    if kind == "ascending":        # every key passes the gate: overflow
        s[:, :nk] = np.arange(nk, dtype=np.float32)
    elif kind == "narrow":         # one binade, neighbours a few ulps apart
        s[:, :nk] = (1.5 + rng.integers(0, 1 << 16, size=(nq, nk)) * 2.0 ** -22).astype(np.float32)
    elif kind == "heavy":          # a distribution that no linear map spreads
        s[:, :nk] = np.exp(np.clip(20 * rng.standard_normal((nq, nk)), -87, 88)).astype(np.float32)
    elif kind == "infs":           # more infinities than k, both signs
        s[:, :nk] = rng.choice([np.inf, -np.inf, 0.0, -0.0, np.nan, 1.0], size=(nq, nk))
    elif kind in ("sparse", "masked", "middle"):  # a few spread scores, the others 0 or -inf
        s[:, :nk] = -np.inf if kind == "masked" else 0.0
        hit = rng.random((nq, nk)) < 0.0002
        v = rng.standard_normal(int(hit.sum()))
        s[:, :nk][hit] = v if kind == "middle" else np.abs(v)
    return torch.from_numpy(s)


def _check(scores, nk, k, offs, starts, gi, gs, sorted_out, rows):
    s = scores.numpy()[rows]
    o = None if offs is None else offs[rows]
    st = None if starts is None else starts[rows]
    ri, rs = orc.topk_select(s, nk, k, o, visible_start=st)
    s0, e0 = orc.visible_ranges(o, st, len(rows), nk)
    for j, t in enumerate(rows):
        check_row_exact(gi[t], gs[t], ri[j], rs[j], int(e0[j] - s0[j]), k, sorted_out)


# block widths follow the rows (1024, 512 and 256 threads from 1, 512 and 1024
# units; one wave for up to 1024 keys), steps the split's length (32768 keys); fewer than 256 rows split
@pytest.mark.parametrize("nq,nk,k,kind", [
    (1, 140001, 100, "normal"),
    (3, 70000, 2048, "ascending"),
    (20, 33000, 7, "narrow"),
    (300, 32767, 64, "ties"),
    (513, 8193, 300, "special"),
    (1025, 4099, 100, "infs"),
    (1024, 40003, 16, "heavy"),
    (130, 257, 300, "normal"),
    (300, 1024, 64, "ascending"),
    (3, 1025, 20, "special"),
    (2000, 255, 16, "infs"),
])
@pytest.mark.parametrize("sorted_out", [False, True])
def test_scores_in_filter_shapes(lib, nq, nk, k, kind, sorted_out):
    scores = _rows(kind, nq, nk, seed=nq + k)
    rng = np.random.default_rng(nk)
    offs = workloads.causal_offsets(nq, nk)
    starts = rng.integers(0, max(1, nk // 3), size=nq).astype(np.int32)  # not multiples of anything
    o, st = torch.from_numpy(offs).cuda(), torch.from_numpy(starts).cuda()
    gi, gs = lt.topk_select(scores.cuda(), k, nk, o, options=lt.make_options(sorted_output=sorted_out,
                                                                             visible_start=st))
    gi, gs = gi.cpu().numpy(), gs.cpu().numpy()
    _check(scores, nk, k, offs, starts, gi, gs, sorted_out, sorted({0, 1 % nq, nq // 2, nq - 1}))


# a workspace with no room for the lists of split rows (here: of the call with
# one split, which is what fewer than 256 rows took before they were split)
@pytest.mark.parametrize("nq,nk,k", [(1, 140001, 100), (60, 66000, 300), (200, 33000, 64)])
def test_scores_in_workspace_for_unsplit_rows(lib, nq, nk, k):
    scores = _rows("normal", nq, nk, seed=nq)
    n = lt.lt_topk_select_workspace_size(nq, nk, k, lt.make_options(key_splits=1))
    assert n <= lt.lt_topk_select_workspace_size(nq, nk, k)
    ws = torch.empty(n + 4096, dtype=torch.uint8, device="cuda")
    ws[n:] = 123
    gi, gs = lt.topk_select(scores.cuda(), k, nk, None, options=lt.make_options(sorted_output=True), workspace=ws[:n])
    assert bool((ws[n:] == 123).all())
    _check(scores, nk, k, None, None, gi.cpu().numpy(), gs.cpu().numpy(), True, sorted({0, nq // 2, nq - 1}))
    with pytest.raises(lt.LiteTopKError):
        lt.topk_select(scores.cuda(), k, nk, None, workspace=ws[:n - 256])


# 256-thread blocks for many short rows, else 1024; k = 2048 and 2049 are the
# last with 4096 sort entries and the first with more
@pytest.mark.parametrize("nq,nk,k", [(600, 3000, 100), (600, 16385, 2048), (40, 16384, 2049), (5, 70001, 8192),
                                     (3, 4097, 4096)])
@pytest.mark.parametrize("kind", ["normal", "ties", "narrow", "heavy", "infs", "const", "sparse", "masked", "middle"])
def test_radix_rows(lib, nq, nk, k, kind):
    scores = _rows(kind, nq, nk, seed=nk + k)
    offs = workloads.causal_offsets(nq, nk)
    offs[0] = min(nk, k + 1)
    gi, gs = lt.topk_radix(scores.cuda(), k, nk, torch.from_numpy(offs).cuda(), sorted_output=True)
    _check(scores, nk, k, offs, None, gi.cpu().numpy(), gs.cpu().numpy(), True, sorted({0, 1, nq - 1}))


# unsorted rows of k > 2048: 8-bit digits alone for more than 256 rows of up to
# 16384 keys and more than 512 of up to 32768
@pytest.mark.parametrize("nq,nk,k", [(256, 5000, 2049), (257, 16384, 2049), (257, 16385, 4096), (513, 32768, 4097),
                                     (513, 32769, 2100), (300, 2050, 2049), (300, 8193, 8192), (300, 16000, 2048)])
@pytest.mark.parametrize("kind", ["normal", "ties", "infs", "middle"])
def test_radix_unsorted_large_k(lib, nq, nk, k, kind):
    scores = _rows(kind, nq, nk, seed=nk + k)
    offs = workloads.causal_offsets(nq, nk)
    offs[0] = k  # no more keys than k
    gi, gs = lt.topk_radix(scores.cuda(), k, nk, torch.from_numpy(offs).cuda())
    _check(scores, nk, k, offs, None, gi.cpu().numpy(), gs.cpu().numpy(), False, sorted({0, 1, nq - 1}))


# the k-th key shared by more keys than the sort slots hold: they are cut by
# index, 64 keys at a time, n / 4096 from 2^18 keys on, and with parts past the
# slots left (2^23) to the general selection
@pytest.mark.parametrize("nq,nk,k", [(600, 16000, 33), (3, 5000, 2048), (2, 600001, 2048), (2, 600001, 5000),
                                     (1, 9000001, 2048)])
@pytest.mark.parametrize("kind", ["const", "sparse", "middle"])
@pytest.mark.parametrize("sorted_out", [False, True])
def test_radix_more_equal_keys_than_slots(lib, nq, nk, k, kind, sorted_out):
    scores = _rows(kind, nq, nk, seed=nk)
    s = scores[0, :nk].numpy()
    assert np.sum(s == np.partition(s, nk - k)[nk - k]) > (12288 if k > 2048 else 3072)
    if nq > 1:
        scores[-1, :nk - 4000] = -5.0  # few of them, at the row's end
    gi, gs = lt.topk_radix(scores.cuda(), k, nk, sorted_output=sorted_out)
    _check(scores, nk, k, None, None, gi.cpu().numpy(), gs.cpu().numpy(), sorted_out, sorted({0, nq - 1}))


# sorted rows whose kept keys no map spreads (more than 128 equal scores, of
# several values): ordered by the sort in LDS. Scores in hand keep their bits
# (both zeros), fused rows report canonical ones.
@pytest.mark.parametrize("nq,nk,k", [(600, 9000, 700), (20, 9000, 700), (20, 40000, 3000), (600, 9000, 2048)])
def test_sorted_rows_of_few_values(lib, nq, nk, k):
    rng = np.random.default_rng(nk + k)
    s = rng.choice([3.0, 2.0, 0.0, -0.0, -1.0], size=(nq, nk), p=[0.02, 0.02, 0.03, 0.03, 0.9]).astype(np.float32)
    assert min(np.unique(np.sort(s[0])[-k:], return_counts=True)[1][1:]) > 128
    scores = torch.from_numpy(s)
    rows = [0, nq // 2, nq - 1]
    for fn in (lambda: lt.topk_select(scores.cuda(), k, nk, options=lt.make_options(sorted_output=True)),
               lambda: lt.topk_radix(scores.cuda(), k, nk, sorted_output=True)):
        gi, gs = fn()
        gi, gs = gi.cpu().numpy(), gs.cpu().numpy()
        _check(scores, nk, k, None, None, gi, gs, True, rows)
        for t in rows:
            np.testing.assert_array_equal(gs[t].view(np.uint32), s[t][gi[t]].view(np.uint32))


# candidate lists per row: one, fewer than a block's waves, more, and four
# times as many (16 waves up to 512 rows, 4 beyond); integer inputs give exact
# scores with many ties
@pytest.mark.parametrize("nq,splits", [(9, 1), (9, 3), (9, 17), (9, 64), (520, 2), (520, 5), (520, 16)])
@pytest.mark.parametrize("k", [50, 2100])
def test_fused_sorted_rows(lib, nq, splits, k):
    x = workloads.exact_inputs(nq, 5000, 64, 128, "bf16", seed=nq + splits)
    d = to_dev(x)
    gi, gs = lt.indexer_topk(d["q"], d["w"], d["keys"], k, d["offsets"],
                             options=lt.make_options(sorted_output=True, key_splits=splits))
    gi, gs = gi.cpu().numpy(), gs.cpu().numpy()
    rows = [0, nq // 2, nq - 1]
    ri, rs, _ = oracle_topk(x, "bf16", k, "dsa", rows=rows)
    for j, t in enumerate(rows):
        check_row_exact(gi[t], gs[t], ri[j], rs[j], int(x["offsets"][t]), k, True)


# launches of few query tiles: splits down to one key tile, rows whose lists
# hold a whole split (no second pass), the fallback without its dense mode (up
# to 128 rows; fewer keys than two chunks: whole rows), and short lists of splits
# that share thresholds
@pytest.mark.parametrize("nq,nk,h,d,dtype,mode,k,opt", [
    (1, 64, 64, 128, "bf16", "dsa", 5, dict()),
    (3, 5000, 64, 128, "fp8", "dsa", 700, dict()),
    (20, 9001, 4, 128, "bf16", "dsa", 300, dict()),
    (50, 3000, 1, 64, "f32", "ip", 100, dict()),
    (50, 3000, 1, 64, "f32", "ip", 100, dict(force_fallback=True)),
    (128, 8191, 64, 128, "bf16", "dsa", 64, dict(force_fallback=True)),
    (129, 8191, 64, 128, "bf16", "dsa", 64, dict(force_fallback=True)),
    (40, 20000, 1, 128, "bf16", "ip", 200, dict(key_splits=4, capacity=400)),
    (300, 4001, 1, 128, "bf16", "dsa", 2000, dict()),  # most lanes pass in most sub-tiles
    (33, 4001, 4, 64, "f32", "dsa", 1000, dict(sample_size=0)),  # no gate at first
])
def test_fused_few_tiles(lib, nq, nk, h, d, dtype, mode, k, opt):
    x = workloads.exact_inputs(nq, nk, h, d, dtype, seed=nq + nk)
    if mode == "ip":
        x["w"] = None
    dev = to_dev(x)
    gi, gs = lt.indexer_topk(dev["q"], dev["w"], dev["keys"], k, dev["offsets"], dev["q_scale"], dev["k_scale"], mode,
                             lt.make_options(sorted_output=True, **opt))
    gi, gs = gi.cpu().numpy(), gs.cpu().numpy()
    rows = sorted({0, nq // 2, nq - 1})
    ri, rs, _ = oracle_topk(x, dtype, k, mode, rows=rows)
    for j, t in enumerate(rows):
        check_row_exact(gi[t], gs[t], ri[j], rs[j], int(x["offsets"][t]), k, True)


# lists of 300 entries for k = 200: every row overflows one and is completed by
# the second pass (row_stats reason 6), over splits that share thresholds
@pytest.mark.parametrize("h,mode", [(1, "ip"), (4, "dsa")])
def test_second_pass_over_shared_thresholds(lib, h, mode):
    nq, nk, k = 40, 20000, 200
    x = workloads.exact_inputs(nq, nk, h, 128, "bf16", seed=5)
    if mode == "ip":
        x["w"] = None
    dev = to_dev(x)
    stats = torch.full((nq, lt.LT_ROW_STATS), -7, dtype=torch.int32, device="cuda")
    gi, gs = lt.indexer_topk(dev["q"], dev["w"], dev["keys"], k, dev["offsets"], mode=mode,
                             options=lt.make_options(sorted_output=True, key_splits=4, capacity=300, row_stats=stats))
    assert bool((stats[:, 2] == 6).all())
    gi, gs = gi.cpu().numpy(), gs.cpu().numpy()
    rows = [0, nq // 2, nq - 1]
    ri, rs, _ = oracle_topk(x, "bf16", k, mode, rows=rows)
    for j, t in enumerate(rows):
        check_row_exact(gi[t], gs[t], ri[j], rs[j], int(x["offsets"][t]), k, True)


# one entry per thread up to 1024 entries a group (512 groups at most); spans
# around what the bitmap of a wide (2^20 keys and some) and of a narrow
# block holds, and keys up to the largest index
@pytest.mark.parametrize("nq,k,group,span,top", [
    (16, 512, 8, 1 << 20, 1 << 20), (16, 512, 8, 1 << 21, 1 << 21), (16, 512, 8, 1000, 2 ** 31 - 1),
    (16, 512, 8, 2 ** 31 - 1, 2 ** 31 - 1), (1100, 64, 2, 200000, 300000), (1100, 64, 2, 400000, 400000),
    (20, 2048, 16, 131072, 131072), (9, 3000, 3, 50000, 50000), (7, 1, 5, 3, 3),
    (18, 128, 8, 1 << 20, 1 << 20), (18, 128, 8, 1 << 21, 1 << 21), (18, 129, 8, 1 << 21, 1 << 21),
    (512, 1023, 1, 131072, 131072), (513, 1023, 1, 131072, 131072)])
def test_union_spans(lib, nq, k, group, span, top):
    rng = np.random.default_rng(k + group)
    idx = (top - span + rng.integers(0, span, size=(nq, k))).astype(np.int32)
    idx[rng.random((nq, k)) < 0.05] = -1
    idx[0, 0], idx[0, -1] = top - span, top - 1  # the first group's span is exact
    u, c, m = lt.dsa_union(torch.from_numpy(idx).cuda(), group)
    ru, rc, rm = orc.dsa_union(idx, group)
    np.testing.assert_array_equal(c.cpu().numpy(), rc)
    np.testing.assert_array_equal(u.cpu().numpy(), ru)
    np.testing.assert_array_equal(m.cpu().numpy().view(np.uint32), rm)


# rows of nearly 2^31 keys, whose last steps pass the largest 32-bit position:
# planted keys (some at the very end), tied background keys below them, k
# within the planted ones and past them
@pytest.mark.parametrize("nk", [2 ** 31 - 1, 2 ** 31 - 20000])
def test_rows_of_2_to_the_31_keys(lib, nk):
    scores = torch.empty(1, 2 ** 31, dtype=torch.float32, device="cuda")
    scores.view(-1, 1024)[:] = -1.0 - torch.arange(1024, device="cuda") / 1024.0
    rng = np.random.default_rng(1)
    at = np.unique(np.concatenate([rng.integers(0, nk, size=400), np.arange(nk - 100, nk)]))
    vals = (10.0 + np.arange(len(at))).astype(np.float32)
    rng.shuffle(vals)
    scores[0, torch.from_numpy(at).cuda()] = torch.from_numpy(vals).cuda()
    order = np.argsort(-vals)
    free = np.setdiff1d(np.arange(0, 2 ** 20, 1024), at)  # background keys of score -1, in order

    def check(i, s, k):
        n = min(k, len(at))
        np.testing.assert_array_equal(i.cpu().numpy()[0, :n], at[order[:n]])
        np.testing.assert_array_equal(s.cpu().numpy()[0, :n], vals[order[:n]])
        np.testing.assert_array_equal(i.cpu().numpy()[0, n:], free[:k - n])
        assert bool((s[0, n:] == -1.0).all())

    check(*lt.topk_radix(scores, 40, nk, sorted_output=True), 40)
    check(*lt.topk_radix(scores, 600, nk, sorted_output=True), 600)
    sample = torch.from_numpy(np.sort(at[:300]).astype(np.int32)).cuda()
    for splits in (0, 1):
        o = lt.make_options(sorted_output=True, sample_keys=sample, key_splits=splits)
        check(*lt.topk_select(scores, 40, nk, options=o), 40)
    o = lt.make_options(sorted_output=True, force_fallback=True)
    check(*lt.topk_select(scores, 600, nk, options=o), 600)
