"""How a launch's tables reach the kernel: among its arguments when they are
small, else through pinned staging that is reused after eight launches.
Either way the results are those of cp_attn_partial_noalloc, which copies its
tables itself and plans the same list, bit for bit.  And launches whose walks
are cut into many or few short pieces, against the oracle, and with NaN and
infinite scores; and merges of every partial count."""

import pytest
import torch

import gpu_cases as gc
from gpu_cases import DEV, Problem
from paper_2609_04774_amd import cpattn as cp

pytestmark = pytest.mark.gpu


def _launch(R, Hq, Hkv, seed, C=1, n_descs=1):
    prob = Problem(R, 0, C, Hq, Hkv, seed)
    dv = prob.dev()
    plan, rows = cp.shard_plan(0, R, C, 0)
    q = dv["q"][torch.as_tensor(rows, device=DEV)].contiguous()
    outs = [gc.alloc_out(plan.n_rows, Hq) for _ in range(2 * n_descs)]
    descs = [cp.make_desc(plan, q, dv["k"], dv["v"], o, lse) for o, lse in outs]
    return descs[:n_descs], descs[n_descs:], outs, n_descs


def _compare(launch, what):
    _, _, outs, n = launch
    for i in range(n):
        assert torch.equal(outs[i][0], outs[n + i][0]) and torch.equal(outs[i][1], outs[n + i][1]), what


# One head per KV head and both chunks of a degree of 1 within a block (R > 1):
# two work items per head.  One descriptor leaves room for 424 words, two for
# 400, 17 for 40.
@pytest.mark.parametrize("rows", [256, 384])
@pytest.mark.parametrize("R,H,n_descs", [(1, 1, 1), (60, 212, 1), (60, 213, 1), (400, 100, 2), (400, 101, 2),
                                         (1, 2, 17), (1, 3, 17), (1, 1, 33)])
def test_tables_on_both_sides_of_the_argument_space(rows, R, H, n_descs):
    try:
        cp.set_workgroup_rows(rows)
        launch = _launch(R, H, H, 11, n_descs=n_descs)
        gc.run_partials(launch[0], H, H)
        cp.attn_partial_noalloc(launch[1], H, H)
        torch.cuda.synchronize()
    finally:
        cp.set_workgroup_rows(0)
    _compare(launch, f"R {R}, heads {H}, descriptors {n_descs}")


def test_staging_is_reused_in_order():
    """Twenty launches of different tables in flight at once, of sizes that
    make the staging slots grow and be written again while earlier launches
    have yet to read theirs."""
    launches, ws = [], []
    for i in range(20):
        H = 425 + 97 * ((7 * i) % 20)
        launches.append((H, _launch(33 + i, H, H, 100 + i)))
        ws.append(gc.new_workspace(launches[-1][1][0], H, H))
    torch.cuda.synchronize()
    torch.cuda._sleep(20_000_000)
    for (H, launch), w in zip(launches, ws):
        cp.attn_partial(launch[0], H, H, w)
    for H, launch in launches:
        cp.attn_partial_noalloc(launch[1], H, H)
    torch.cuda.synchronize()
    for H, launch in launches:
        _compare(launch, f"{H} heads")


@pytest.mark.parametrize("H", [8, 500])
def test_a_captured_launch_replays(H):
    launch = _launch(200, H, H, 21)
    ws = gc.new_workspace(launch[0], H, H)
    other = _launch(77, 8, 8, 22)
    other_ws = gc.new_workspace(other[0], 8, 8)
    for _ in range(8):  # every staging slot is allocated before the capture
        cp.attn_partial(launch[0], H, H, ws)
    cp.attn_partial_noalloc(launch[1], H, H)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        cp.attn_partial(launch[0], H, H, ws)
    for _ in range(3):
        launch[2][0][0].zero_()
        launch[2][0][1].zero_()
        graph.replay()
        torch.cuda.synchronize()
        _compare(launch, f"replay, {H} heads")
        cp.attn_partial(other[0], 8, 8, other_ws)
    torch.cuda.synchronize()


def test_a_captured_launch_replays_after_staged_ones():
    """A graph whose launch has tables beyond the argument space, replayed
    after more staged launches than there are slots, larger ones among them."""
    H = 500
    launch = _launch(200, H, H, 23)
    ws = gc.new_workspace(launch[0], H, H)
    others = []
    for i in range(10):
        h = 430 + 60 * i
        others.append((h, _launch(50 + i, h, h, 200 + i)))
        others[-1] += (gc.new_workspace(others[-1][1][0], h, h),)
    cp.attn_partial_noalloc(launch[1], H, H)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        cp.attn_partial(launch[0], H, H, ws)
    for _ in range(3):
        for h, other, w in others:
            cp.attn_partial(other[0], h, h, w)
        torch.cuda.synchronize()
        ws.zero_()
        launch[2][0][0].zero_()
        launch[2][0][1].zero_()
        graph.replay()
        torch.cuda.synchronize()
        _compare(launch, "replay")


# (L, P, C, Hq, Hkv, rank): pieces of three or four tiles; six and more per
# item; 64 per item (a wave merges each row); pieces that some rows see no key
# of; one and three query rows; a 384-row list of a few pieces per item; head
# groups that no XCD count divides.
@pytest.mark.parametrize("L,P,C,Hq,Hkv,rank", [
    (1024, 0, 2, 8, 2, 0), (2900, 880, 1, 8, 2, 0), (6073, 6016, 8, 8, 2, 3), (2049, 2048, 1, 4, 1, 0),
    (4099, 4096, 1, 16, 1, 0), (4700, 4400, 1, 32, 8, 0), (1500, 608, 2, 24, 3, 1), (1203, 1200, 2, 8, 8, 0)])
def test_cut_walks_match_oracle(L, P, C, Hq, Hkv, rank):
    prob = Problem(L, P, C, Hq, Hkv, 31)
    o, lse, plan, _ = prob.gpu_rank(rank)
    Or, Lr = prob.oracle_rank(rank)
    gc.compare(gc.f64(o), gc.f64(lse), Or, Lr, f"rank {rank} of {C}")


def test_a_smaller_workspace_gets_fewer_pieces():
    """A workspace below the sizing call's figure, down to the tables of an
    uncut list, is still taken (with longer pieces); below that it is refused."""
    prob = Problem(2348, 2048, 1, 8, 2, 33)
    dv = prob.dev()
    plan, _ = cp.shard_plan(prob.P, prob.R, 1, 0)
    o, lse = gc.alloc_out(plan.n_rows, 8)
    desc = cp.make_desc(plan, dv["q"], dv["k"], dv["v"], o, lse, dv["kc"], dv["vc"], dv["bt"])
    full = cp.workspace_size([desc], 8, 2)
    Or, Lr = prob.oracle_rank(0)
    assert full > 1 << 20
    for size in (full, full - 256, full // 2, 4096):
        ws = torch.empty(size, dtype=torch.uint8, device=DEV)
        o.fill_(float("nan"))
        cp.attn_partial([desc], 8, 2, ws)
        torch.cuda.synchronize()
        gc.compare(gc.f64(o), gc.f64(lse), Or, Lr, f"{size} bytes")
    with pytest.raises(cp.CpError) as e:
        cp.attn_partial([desc], 8, 2, torch.empty(256, dtype=torch.uint8, device=DEV))
    assert e.value.status == cp.CP_ERR_CAPACITY


@pytest.mark.parametrize("n", range(1, 17))
def test_merge_of_every_partial_count(n):
    """Each partial count has its own kernel up to eight; 31 and 33 rows end a
    block and a two-row group short.  fp32: weights within 2^-21 (expf, one
    division) and n products, |O| below 6: 1e-5; bf16: half an ulp more."""
    g = torch.Generator().manual_seed(50 + n)
    for n_tok, H in ((31, 1), (11, 3), (100, 5)):
        o = [torch.randn(n_tok, H, 128, generator=g) for _ in range(n)]
        lse = [torch.randn(n_tok, H, generator=g) * 4 for _ in range(n)]
        for i in range(n):
            lse[i][torch.rand(n_tok, H, generator=g) < 0.2] = float("-inf")
        w = torch.stack(lse).double()
        L = torch.logsumexp(w, 0)
        ref = sum(torch.nan_to_num((w[i] - L).exp())[..., None] * o[i].double() for i in range(n))
        od, ld = [x.to(DEV) for x in o], [x.to(DEV) for x in lse]
        O, Ob = torch.empty(n_tok, H, 128, device=DEV), torch.empty(n_tok, H, 128, dtype=torch.bfloat16, device=DEV)
        Lo = torch.empty(n_tok, H, device=DEV)
        cp.attn_merge(od, ld, O, Lo)
        cp.attn_merge(od, ld, Ob)
        torch.cuda.synchronize()
        live = torch.isfinite(L)
        assert torch.equal(torch.isfinite(Lo.cpu()), live)
        assert float((Lo.cpu().double() - L)[live].abs().max()) < 5e-6
        assert float((O.cpu().double() - ref).abs().max()) < 1e-5
        assert bool(((Ob.cpu().double() - ref).abs() <= ref.abs() * 2.0 ** -8 + 1e-5).all())


# (L, P, C, Hq, Hkv, cut): a launch whose walks are cut (few key tiles a piece;
# a cached prefix; a wave per merged row) or, with many heads, not.
@pytest.mark.parametrize("L,P,Hq,Hkv,cut", [(1024, 0, 32, 8, True), (1348, 1248, 32, 8, True),
                                            (4099, 4096, 16, 1, True), (600, 0, 512, 128, False)])
@pytest.mark.parametrize("bad", [float("nan"), float("inf")])
def test_a_poisoned_score_shows_cut_or_not(L, P, Hq, Hkv, cut, bad):
    """A key or a query row that makes scores NaN (+inf does by inf - inf)
    leaves O = NaN and LSE = -inf in every row that meets it, whether or not
    the row's walk is cut.  Rows that do not meet it keep their values, but for
    the running max that P is rounded against (bf16, half an ulp each way)."""
    prob = Problem(L, P, 1, Hq, Hkv, 41)
    clean, clean_lse, plan, _ = prob.gpu_rank(0)
    dv = prob.dev()
    desc = cp.make_desc(plan, dv["q"], dv["k"], dv["v"], clean, clean_lse, dv.get("kc"), dv.get("vc"), dv.get("bt"))
    assert (cp.workspace_size([desc], Hq, Hkv) > 1 << 20) == cut
    R, G, pos = L - P, Hq // Hkv, 2 * (L - P) // 3
    dv["k"][pos, 0, 5] = bad  # KV head 0's key at suffix index pos
    dv["q"][R // 2, Hq - 1] = float("nan")
    o, lse, _, _ = prob.gpu_rank(0)
    met = torch.zeros(R, Hq, dtype=torch.bool, device=DEV)
    met[pos:, :G] = True
    met[R // 2, Hq - 1] = True
    hit = met.clone()
    if bad == float("inf"):  # a score of -inf is a key of weight 0
        hit[pos:, :G] &= ~(dv["q"][pos:, :G, 5] < 0)
    assert bool(o[hit].isnan().all()) and bool(torch.isneginf(lse[hit]).all())
    assert bool(torch.isfinite(o[~hit]).all()) and bool(torch.isfinite(lse[~hit]).all())
    assert float((o - clean)[~met].abs().max()) <= 2.0 ** -8 * float(dv["v"].float().abs().max())
    assert float((lse - clean_lse)[~met].abs().max()) <= 1e-5
