"""How launches deal their work: sizes at which the last round of a Refine
launch holds a few row blocks only, so that they are cut into candidate slices
and shared by all SIMDs, and batches whose sequences hold different numbers of
groups on the proxy path."""
import numpy as np
import pytest
import torch

import oracle
import paper_2607_24593_amd as pv
from gpu_util import dev, host, say
from parity import check_pivot
from test_gpu_layout import _groups, check_batch, run_batch
from workload.gen import make_prefill

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def inputs():
    return {f: make_prefill(7400, f, seed=81, threads=8) for f in ("fp8", "bf16")}


# fp8 blocks hold 4 members, bf16 blocks 2: groups of 4 make 1 or 2 blocks a group
@pytest.mark.parametrize("fmt,p0,n_q,g,c,topk", [
    ("fp8", 2100, 4 * 1024, 4, 1024, 300),       # 1024 blocks: one whole round, none cut
    ("fp8", 2100, 4 * 1024 + 1, 4, 1024, 300),   # one block of one member past it
    ("fp8", 2100, 4 * 1300 - 3, 4, 2040, 300),   # a quarter of a round past it, ragged candidate tail
    ("fp8", 2100, 5001, 8, 1000, 300),           # two blocks a group, ragged last group of one
    ("fp8", 2100, 2 * 600, 2, 1024, 300),        # less than a round (2-row blocks), all cut
    ("bf16", 2100, 2 * 1100 + 1, 2, 1016, 300),  # 1101 blocks
    ("bf16", 2100, 4 * 513, 4, 1024, 300),       # 1026 blocks of two a group
])
def test_refine_tail_blocks(inputs, fmt, p0, n_q, g, c, topk):
    """Sampled groups, the last ones (the cut blocks) among them, against the oracle."""
    x, n_k, ng = inputs[fmt], p0 + n_q, -(-n_q // g)
    say("refine tail", fmt, n_q, g, c)
    qs = None if x.q_scale is None else x.q_scale[p0:n_k]
    ks = None if x.k_scale is None else x.k_scale[:n_k]
    cand = torch.full((1, ng, c), -7, dtype=torch.int32, device="cuda")
    idx = pv.pivot_group_index(dev(x.q[p0:n_k]), dev(qs), dev(x.w[p0:n_k]), dev(x.k[:n_k]), dev(ks), p0, n_k, topk,
                               mode=pv.PIVOT_REFINE, g=g, c=c, out_cand=cand)
    rng = np.random.default_rng(3)
    groups = sorted({0, 1, ng - 3, ng - 2, ng - 1} | set(int(v) for v in rng.integers(0, ng, 8)))
    check_pivot(fmt, x.q[p0:n_k], qs, x.w[p0:n_k], p0, x.k[:n_k], ks, n_k, mode=oracle.REFINE, g=g, c=c, topk=topk,
                dense_below=-1, gpu_idx=host(idx), gpu_cand=host(cand)[0], groups=groups, label="tail")


def test_refine_ragged_batch_matches_single_calls(inputs):
    """Packed runs with different numbers of proxy groups (one sequence wholly
    on the guardrail, one empty, one of a single query) give each sequence the
    sets of its own call."""
    x, g, c, topk = inputs["fp8"], 4, 1024, 300
    runs = [(0, 900), (1500, 2303), (3000, 0), (5000, 1), (2000, 2401)]  # (first position, queries)
    cu = np.concatenate([[0], np.cumsum([n for _, n in runs])])
    rows = np.concatenate([np.arange(p, p + n) for p, n in runs])
    lens = [p + max(n, 1) for p, n in runs]
    k = torch.zeros(len(runs), max(lens), 128, dtype=torch.uint8, device="cuda")
    ks = torch.ones(len(runs), max(lens), device="cuda")
    for b, n in enumerate(lens):
        k[b, :n], ks[b, :n] = dev(x.k[:n]), dev(x.k_scale[:n])
    say("refine ragged batch", runs)
    got = host(pv.pivot_group_index_layout(dev(x.q[rows]), dev(x.q_scale[rows]), dev(x.w[rows]), k, ks,
                                           [p for p, _ in runs], lens, topk, pv.make_layout(cu), pv.PIVOT_REFINE, g, c))
    for b, (p, n) in enumerate(runs):
        if n == 0:
            continue
        e = p + n
        one = host(pv.pivot_group_index(dev(x.q[p:e]), dev(x.q_scale[p:e]), dev(x.w[p:e]), dev(x.k[:e]),
                                        dev(x.k_scale[:e]), p, e, topk, mode=pv.PIVOT_REFINE, g=g, c=c))
        assert np.array_equal(np.sort(got[cu[b]:cu[b + 1]], 1), np.sort(one, 1)), (b, p, n)


@pytest.mark.parametrize("topk", [1, 200, 2048, 3900, 4095])
@pytest.mark.parametrize("scale", [1.0, 1e3, 0.0])
def test_member_select_heavy_tails(topk, scale):
    """Member rows whose largest scores are far past the others (Pareto keys,
    some scaled up further; scale 0: a third of the keys are zero, so their
    scores are equal and lie inside the cut range), selected from 4096 slots:
    the same sets as the fused path, whose select does not use value ranges."""
    x = make_prefill(6000, "fp8", seed=83, boost=("pareto", 0.02, 0.7), threads=8)
    x.k_scale = x.k_scale.copy()
    x.k_scale[np.arange(6000) % (97 if scale > 0 else 3) == 0] *= np.float32(scale)
    p0, g, c = 5000, 4, 4096
    args = (dev(x.q[p0:]), dev(x.q_scale[p0:]), dev(x.w[p0:]), dev(x.k), dev(x.k_scale), p0, 6000, topk)
    say("heavy tails", topk, scale)
    a, b = (host(pv.pivot_group_index_opts(*args, mode=pv.PIVOT_REFINE, g=g, c=c, refine_path=path))
            for path in (pv.PIVOT_REFINE_SPLIT, pv.PIVOT_REFINE_FUSED))
    assert np.array_equal(np.sort(a, 1), np.sort(b, 1))


@pytest.mark.parametrize("fmt", ["fp8", "bf16"])
@pytest.mark.parametrize("page", [16, 256, 4096])
@pytest.mark.parametrize("g", [1, 2, 3, 20])
def test_short_segments_paged_equal_contiguous(inputs, fmt, page, g):
    """Few short sequences take key segments of 128 or 256 keys, smaller than a
    page or a whole number of pages; limits fall on, before and after a segment
    edge.  Paged and contiguous keys give the same sets, and both the sets of a
    call on each sequence alone (whose segments may differ)."""
    x, lens, topk = inputs[fmt], [127 + g, 128 + g, 129 + g, 1024, 2049, 7391], 100
    runs = [(n - g, g) for n in lens]
    rows = np.concatenate([np.arange(p, p + n) for p, n in runs])
    cu = np.concatenate([[0], np.cumsum([n for _, n in runs])])
    need = [-(-n // page) for n in lens]
    order = np.random.default_rng(page + g).permutation(sum(need)).astype(np.int32)
    table = np.zeros((len(lens), max(need)), np.int32)
    pool = np.zeros((sum(need), page, 128), x.k.dtype)
    pool_s = np.ones((sum(need), page), np.float32)
    first = 0
    for b, n in enumerate(lens):
        mine = order[first:first + need[b]]
        first += need[b]
        table[b, :need[b]] = mine
        whole, sc = np.zeros((need[b] * page, 128), x.k.dtype), np.ones(need[b] * page, np.float32)
        whole[:n] = x.k[:n]
        if fmt == "fp8":
            sc[:n] = x.k_scale[:n]
        pool[mine], pool_s[mine] = whole.reshape(-1, page, 128), sc.reshape(-1, page)
    q, w = dev(x.q[rows]), dev(x.w[rows])
    qs = dev(x.q_scale[rows]) if fmt == "fp8" else None
    ps = dev(pool_s.reshape(-1)) if fmt == "fp8" else None
    lay = pv.make_layout(cu, dev(table), page, sum(need) * page)
    say("short segments", fmt, page, g)
    args = (q, qs, w, dev(pool.reshape(-1, 128)), ps, [p for p, _ in runs], lens, topk, lay)
    dense = np.sort(host(pv.pivot_dense_index_layout(*args)), 1)
    refine = np.sort(host(pv.pivot_group_index_layout(*args, pv.PIVOT_REFINE, g, 2 * topk)), 1)
    for b, (p, n) in enumerate(runs):
        e = p + n
        one = (dev(x.q[p:e]), dev(x.q_scale[p:e]) if fmt == "fp8" else None, dev(x.w[p:e]), dev(x.k[:e]),
               dev(x.k_scale[:e]) if fmt == "fp8" else None, p, e, topk)
        assert np.array_equal(dense[cu[b]:cu[b + 1]], np.sort(host(pv.pivot_dense_index(*one)), 1)), b
        one_r = host(pv.pivot_group_index(*one, mode=pv.PIVOT_REFINE, g=g, c=2 * topk))
        assert np.array_equal(refine[cu[b]:cu[b + 1]], np.sort(one_r, 1)), b


@pytest.mark.parametrize("short_rows", [0, 1, 40, 280])  # of 300 proxies; 16 rows are the least a call takes
def test_score_rows_borrow_idle_workspace(short_rows):
    """A score region a few rows too small: the score tile reaches into the
    regions that are idle meanwhile (the split select's scratch of a dense call;
    Refine's member scores too).  The sets are those of the full workspace, and
    nothing past it is written."""
    x = make_prefill(17000, "fp8", seed=84, threads=8)
    p0, n_q, topk, g, c = 16100, 900, 300, 3, 1000
    args = (dev(x.q[p0:p0 + n_q]), dev(x.q_scale[p0:p0 + n_q]), dev(x.w[p0:p0 + n_q]), dev(x.k), dev(x.k_scale), p0,
            17000, topk)
    row = ((17000 + 63) // 64 | 1) * 64 * 2
    say("borrowed rows", short_rows)
    a = pv.make_args(*args, torch.empty(n_q, topk, dtype=torch.int32, device="cuda"))
    for kind in ("dense", "refine"):
        need = pv.pivot_workspace_size(a) if kind == "dense" else \
            pv.pivot_group_workspace_size(a, pv.group_opts(pv.PIVOT_REFINE, g, c))
        call = (lambda ws: pv.pivot_dense_index(*args, ws=ws)) if kind == "dense" else \
            (lambda ws: pv.pivot_group_index(*args, pv.PIVOT_REFINE, g, c, ws=ws))
        full = np.sort(host(call(torch.empty(need, dtype=torch.uint8, device="cuda"))), 1)
        less = need - short_rows * row
        buf = torch.full((less + 4096,), 0x5A, dtype=torch.uint8, device="cuda")
        assert np.array_equal(np.sort(host(call(buf[:less])), 1), full), kind
        assert bool((buf[less:] == 0x5A).all()), kind


def _score_launches(call):
    pv.pivot_profile_begin(["score"])
    try:
        out = call()
    finally:
        prof = pv.pivot_profile_end()
    return out, prof["score"][0]


@pytest.mark.parametrize("fmt,p0,n_q,g,c,topk,window", [
    ("fp8", 0, 6001, 4, 2048, 500, 0),     # guardrail rows and proxies in one scoring and one select launch
    ("fp8", 0, 7000, 8, 4096, 2048, 4),    # the shared window's shifted limits beside unshifted ones
    ("fp8", 0, 6001, 2, 900, 200, 0),      # member scores smaller than the score tiles
    ("bf16", 0, 2047, 3, 512, 200, 0),     # 171 guardrail groups, the last one cut by the threshold
    ("bf16", 900, 1200, 2, 1024, 300, 3),  # 124 dense rows
    ("fp8", 500, 560, 4, 520, 100, 0),     # 20 dense rows
    ("fp8", 500, 540, 4, 990, 100, 0),     # 12 proxies: apart
])
@pytest.mark.parametrize("mode", ["reuse", "refine"])
def test_guardrail_beside_proxies(inputs, fmt, p0, n_q, g, c, topk, window, mode):
    """Calls with groups on both sides of the guardrail against the oracle (the
    sampled groups include both sides of it), and the same sets with the least
    workspace, in which the two sets of score rows are apart unless the idle
    regions (Refine's member scores) hold them together; the count of scoring
    launches says which."""
    if window and mode == "reuse":
        pytest.skip("the window applies to Refine")
    x, n_k, ng = inputs[fmt], p0 + n_q, -(-n_q // g)
    say("guardrail", fmt, n_q, g, c, mode)
    qs = None if x.q_scale is None else x.q_scale[p0:n_k]
    ks = None if x.k_scale is None else x.k_scale[:n_k]
    args = (dev(x.q[p0:n_k]), dev(qs), dev(x.w[p0:n_k]), dev(x.k[:n_k]), dev(ks), p0, n_k, topk)
    m = pv.PIVOT_REFINE if mode == "refine" else pv.PIVOT_REUSE
    cand = torch.full((1, ng, c), -7, dtype=torch.int32, device="cuda") if mode == "refine" else None
    got, launches = _score_launches(
        lambda: host(pv.pivot_group_index_opts(*args, m, g, c, window=window, out_cand=cand)))
    edge = max(0, -(-(c - p0) // g))
    dense, proxies, sb = edge * g, ng - edge, 2 if fmt == "fp8" else 4
    o = pv.group_opts(m, g, c, window=window)
    lent = ng * g * pv.pivot_cand_width(o) * sb if mode == "refine" else 0
    both = (proxies * n_k + dense * min(n_k, p0 + dense)) * sb
    if min(dense, proxies) < 16:
        assert launches == 2
    elif 1.1 * both < lent + max(dense, proxies) * n_k * sb:
        assert launches == 1, (lent, both)
    if not window:
        groups = sorted({0, edge - 1, edge, edge + 1, ng - 1} | set(range(0, ng, max(1, ng // 7))))
        check_pivot(fmt, x.q[p0:n_k], qs, x.w[p0:n_k], p0, x.k[:n_k], ks, n_k,
                    mode=oracle.REFINE if mode == "refine" else oracle.REUSE, g=g, c=c, topk=topk, dense_below=-1,
                    gpu_idx=got, gpu_cand=None if cand is None else host(cand)[0],
                    groups=[j for j in groups if 0 <= j < ng], label="guardrail")
    a = pv.make_args(*args, torch.empty(n_q, topk, dtype=torch.int32, device="cuda"))
    need = pv.pivot_group_workspace_size(a, o)
    row = ((n_k + 63) // 64 | 1) * 64 * sb
    least = need - max(0, max(dense, proxies) - 16) * row  # a score region of 16 rows
    small = torch.empty(least, dtype=torch.uint8, device="cuda")
    one, launches = _score_launches(lambda: host(pv.pivot_group_index_opts(*args, m, g, c, window=window, ws=small)))
    assert np.array_equal(np.sort(one, 1), np.sort(got, 1))
    if lent < 0.9 * both:
        assert launches > 1, (lent, both)


@pytest.mark.parametrize("paged", [False, True])
@pytest.mark.parametrize("fmt,mode,window", [("bf16", "reuse", 0), ("bf16", "refine", 0), ("bf16", "refine", 8),
                                             ("fp8", "refine", 8)])
def test_packed_guardrail_beside_proxies(inputs, fmt, mode, window, paged):
    """Packed requests of which one lies on both sides of the guardrail, one wholly
    past it and one wholly below, scored in one launch: contiguous and paged keys,
    with and without the shared window, every request against the oracle."""
    specs = [(1100, 0, 1100), (5000, 3000, 517), (2500, 0, 64)]  # (keys, first position, queries)
    g, c, topk, xs = 4, 256, 128, [inputs[fmt]] * 3
    (idx, cand, cu), launches = _score_launches(
        lambda: run_batch(xs, specs, mode, topk, g, c, paged=paged, page=32, window=window, seed=3))
    assert launches == 1
    check_batch(xs, specs, mode, topk, idx, cand, cu, g, c, window=window,
                groups=_groups(specs, g, c, np.random.default_rng(6)))
