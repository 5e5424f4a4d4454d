"""A layer step whose selection copies the kept rows itself, against the four calls (whose gather kernel copies them): the same
bits, for shares of one row, none and many, K or V alone, strided and misaligned destinations, small and large tables."""
import pytest
import torch

from helpers import STEP_COPY

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("form", ["both", "k", "v", "strided", "misaligned"])
@pytest.mark.parametrize("shape,lens,ks,tail,tensors,parts,units", STEP_COPY)
def test_rows_copied_by_the_selection(shape, lens, ks, tail, tensors, parts, units, form):
    """(The host tests hold `parts` and `units`, of the form with that many tensors, to what the library decides.)"""
    from paper_2604_06746_amd import binding as B
    from paper_2604_06746_amd.sweep import LayerSweep
    Hq, G, d, dtype = shape
    dtype, w = (torch.bfloat16 if dtype == "bf16" else torch.float32), 8
    sw = LayerSweep(Hq, G, d, w, dtype, lens, ks)
    g = torch.Generator(device="cuda")
    g.manual_seed(sum(lens) + tail)
    q = torch.randn(len(lens), Hq, w, d, generator=g, device="cuda").to(dtype)
    k = torch.randn(G, sum(lens), d, generator=g, device="cuda").to(dtype)
    v = torch.randn(G, sum(lens), d, generator=g, device="cuda").to(dtype)
    rows = [x + tail for x in ks]
    total = sum(rows)

    def dst():
        if form == "strided":
            return torch.full((G, 2 * total + 3, 2 * d), -7.0, device="cuda", dtype=dtype)[:, :total, :d]
        if form == "misaligned":
            return torch.full((G * total * d + 2,), -7.0, device="cuda", dtype=dtype)[2:].view(G, total, d)
        return torch.full((G, total, d), -7.0, device="cuda", dtype=dtype)
    want_k, want_v, got_k, got_v = (dst() for _ in range(4))
    cen = torch.rand(sum(lens), generator=g, device="cuda")
    cen2 = cen.clone()
    idx = torch.full((total,), -1, dtype=torch.int32, device="cuda")
    B.structkv_score_layer(sw.shape, q, k, sw.cu, sw.indeg, sw.entropy, sw.entropy_per_head, sw.workspace)
    B.structkv_accumulate_centrality(cen, sw.indeg, 0.9, 1.0 / w)
    B.structkv_select_topk(sw.indeg, sw.cu, ks, tail, idx, sw.topk_workspace)
    B.structkv_gather_kv(k if form != "v" else None, v if form != "k" else None, want_k if form != "v" else None,
                         want_v if form != "k" else None, sw.cu, rows, idx)
    indeg, ent, enth = torch.full_like(sw.indeg, -1), torch.full_like(sw.entropy, -1), torch.full_like(sw.entropy_per_head, -1)
    got_idx = torch.full_like(idx, -1)
    sw.workspace.fill_(0xA5)
    B.structkv_layer_step(sw.shape, q, k, v, sw.cu, ks, tail, indeg, cen2, 0.9, 1.0 / w, ent, enth, got_idx,
                          got_k if form != "v" else None, got_v if form != "k" else None, sw.workspace)
    torch.cuda.synchronize()
    assert torch.equal(got_idx, idx)
    for a, b in ((got_k, want_k), (got_v, want_v)):
        base = (lambda x: x._base if x._base is not None else x)   # (the gaps of a strided destination too)
        assert torch.equal(base(a), base(b))
    assert torch.equal(indeg, sw.indeg) and torch.equal(cen2, cen) and torch.equal(ent, sw.entropy) and torch.equal(enth, sw.entropy_per_head)


def _scores(kind, n, g):
    x = torch.randn(n, generator=g, device="cuda")
    return {"spread": lambda: torch.exp(0.5 * x) / n, "signed": lambda: torch.where(x.abs() < 0.5, -0.0 * x.abs(), x),
            "close": lambda: 1.0 + 1e-4 * x, "plateau": lambda: torch.where(x.abs() < 0.13, 0.0 * x, x),
            "equal": lambda: torch.full_like(x, 0.25),
            "two": lambda: torch.where(x > 0, 3.0, 2.0), "zeros": lambda: torch.where(x > 1, x, torch.zeros_like(x))}[kind]()


@pytest.mark.parametrize("kind", ["spread", "signed", "close", "plateau", "equal", "two", "zeros"])
@pytest.mark.parametrize("lens,tail", [((8193,), 0), ((8200, 100), 8), ((9217, 16384, 12), 0), ((16384 + 32,), 32), ((16385,), 0),
                                       ((8193, 5) * 5 + (16000,), 0), ((8193,) * 28, 0), ((8193,) * 29, 0),
                                       ((17000, 8, 9000) * 21 + (33000,), 8)])
def test_selection_of_up_to_16384_scores(lens, tail, kind):
    """One launch behind the histogram, and the first size that takes two: lists of candidates, a tenth of the scores equal (a list of
    ties), too many for a list.  More sequences than the small table holds; as many workgroups (9 a sequence) as one launch takes, and more;
    the most sequences, some of which have no workgroup, odd and even numbers of shares."""
    from paper_2604_06746_amd import binding as B
    g = torch.Generator(device="cuda")
    g.manual_seed(sum(lens))
    scores = torch.cat([_scores(kind, n, g) for n in lens])
    cu = [sum(lens[:i]) for i in range(len(lens) + 1)]
    ws = torch.empty(B.structkv_workspace_bytes(None, len(lens), cu[-1]), dtype=torch.uint8, device="cuda")
    for share in (0.0, 1e-4, 0.03, 0.5, 1.0):
        ks = [int(share * (n - tail)) for n in lens]
        idx = torch.full((sum(ks) + tail * len(lens) + 1,), -1, dtype=torch.int32, device="cuda")
        ws.fill_(0x5A)
        B.structkv_select_topk(scores, cu, ks, tail, idx, ws)
        want = []
        for b, n in enumerate(lens):
            order = torch.argsort(scores[cu[b]:cu[b] + n - tail] + 0.0, descending=True, stable=True)[:ks[b]]
            want += [order.sort().values, torch.arange(n - tail, n, device="cuda")]
        torch.cuda.synchronize()
        assert torch.equal(idx[:-1].long(), torch.cat(want)) and int(idx[-1]) == -1, (share, kind)
