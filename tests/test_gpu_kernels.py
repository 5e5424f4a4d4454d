"""GPU parity of single kernels at the sizes where they can go wrong: edges of tiles, remainders, the smallest and
largest of their ranges.  Against the fp64 CPU oracle, through the C ABI.

Tolerances: fp32 inputs 1e-5 relative (a dot product of up to 256 fp32 terms is good to a few 1e-7 of its absolute
terms, the exponent to as much absolutely, 2^x to 1 ulp, sums of up to 1e3 of those add 1e-6); bf16 inputs 1e-3, the
bar of the other parity tests.  Selections and copies are exact.
"""
import numpy as np
import pytest
import torch

from helpers import LONG_CHUNKS, LONG_CHUNKS_PIVOT, assert_close_floor, assert_entropy, to_oracle_array

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def B():
    from paper_2604_06746_amd import binding
    return binding


@pytest.fixture(scope="module")
def sweep_mod():
    from paper_2604_06746_amd import sweep
    return sweep


def _randn(*shape, dtype, seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    return torch.randn(*shape, generator=g, device="cuda").to(dtype)


def _score(B, sw, q, k, two_pass):
    """The scoring call; two_pass: its four kernels one by one, which never go through the one launch of short sequences."""
    if not two_pass:
        sw.score(q, k)
        return
    for step in (1, 2, 4, 8):
        B.structkv_debug_score_steps(sw.shape, q, k, sw.cu, sw.indeg, sw.entropy, sw.entropy_per_head, sw.workspace, step)


def _check_scores(sweep_mod, oracle, Hq, G, d, w, dtype, causal, lens, pad=0, scale=0.0, two_pass=False, late=0.0):
    """Score one layer and compare in-degree and entropies; pad: extra elements between key rows (odd strides); late: from this
    share of every sequence on its keys are 24 times larger."""
    total = sum(lens)
    sw = sweep_mod.LayerSweep(Hq, G, d, w, dtype, lens, [0] * len(lens), causal=causal, scale=scale)
    q = _randn(len(lens), Hq, w, d, dtype=dtype, seed=1)
    k = _randn(G, total, d + pad, dtype=dtype, seed=2)[:, :, :d]
    if late:
        for b in range(len(lens)):
            k[:, sw.cu[b] + int(late * lens[b]):sw.cu[b + 1], :] *= 24.0
    sw.indeg.fill_(-7.0)
    _score(sweep_mod.B, sw, q, k, two_pass)
    torch.cuda.synchronize()
    D, ent, ent_h, _ = oracle.score_layer(to_oracle_array(q), to_oracle_array(k), Hq, G, d, w, lens, causal=causal, scale=scale)
    tol = 1e-5 if dtype == torch.float32 else 1e-3
    assert_close_floor(sw.indeg.cpu().numpy(), D, tol, "indeg")
    assert_entropy(sw.entropy.cpu().numpy()[:len(lens)], ent, tol)
    assert_entropy(sw.entropy_per_head.cpu().numpy()[:len(lens)], ent_h, tol)


# head_dim around the padded sizes 64 / 128 / 256, rows around the 32-row waves (one, two, three and more row-chunks),
# keys around the 32-key tiles and the 1024-key workgroups, aligned and odd strides
@pytest.mark.parametrize("Hq,G,d,w,lens,pad", [(1, 1, 1, 1, [1], 0), (2, 2, 64, 32, [31, 33], 0), (4, 2, 65, 17, [32, 97], 0),
                                               (4, 1, 128, 16, [1025], 0), (6, 2, 128, 32, [2049, 5], 4), (8, 1, 40, 33, [4097], 1),
                                               (2, 1, 256, 40, [300], 0), (3, 3, 200, 8, [64, 1, 700], 3)])
@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("causal", [False, True])
@pytest.mark.parametrize("two_pass", [False, True])
def test_fp32_matrix_scoring_kernels(sweep_mod, oracle, Hq, G, d, w, lens, pad, dtype, causal, two_pass):
    if causal:
        lens = [max(n, w) for n in lens]
    _check_scores(sweep_mod, oracle, Hq, G, d, w, dtype, causal, lens, pad, two_pass=two_pass)


# causal windows that are no multiple of the 32-row blocks: heads straddle row blocks and waves; one- and four-wave workgroups
@pytest.mark.parametrize("Hq,G,d,w", [(8, 2, 128, 1), (8, 2, 128, 7), (32, 8, 128, 8), (4, 4, 64, 33), (10, 2, 64, 24), (8, 2, 128, 40),
                                      (2, 1, 128, 100), (3, 1, 64, 40)])
@pytest.mark.parametrize("two_pass", [False, True])
def test_causal_windows_on_the_bf16_kernels(sweep_mod, oracle, Hq, G, d, w, two_pass):
    _check_scores(sweep_mod, oracle, Hq, G, d, w, torch.bfloat16, True, [w, w + 1, 257, 64 + w, 1111], two_pass=two_pass)


# the two-pass bf16 kernels on sequences that ordinary calls score in one launch: one and two row blocks, one and four waves,
# both head sizes; keys late in a chunk that outgrow its first tile's reference by far (pass 1 runs it again)
@pytest.mark.parametrize("Hq,G,d,w,lens", [(8, 2, 128, 8, [1234, 77]), (4, 2, 128, 32, [1700]), (4, 4, 64, 32, [1111]), (2, 2, 64, 64, [900, 45]),
                                           (6, 2, 128, 32, [1700, 45]), (10, 2, 64, 24, [1203]), (8, 2, 128, 40, [999]),
                                           (8, 2, 64, 64, [1500])])
@pytest.mark.parametrize("causal", [False, True])
@pytest.mark.parametrize("late", [0.0, 0.4])
def test_two_pass_kernels_on_short_sequences(sweep_mod, oracle, Hq, G, d, w, lens, causal, late):
    if causal:
        lens = [max(n, w) for n in lens]
    _check_scores(sweep_mod, oracle, Hq, G, d, w, torch.bfloat16, causal, lens, two_pass=True, late=late)


# one scoring launch: keys with gaps between the rows, another scale than 1/sqrt(head_dim), the table of 64 sequences
@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("causal", [False, True])
@pytest.mark.parametrize("Hq,G,d,w,lens,pad,scale", [(8, 2, 128, 8, [700, 33], 8, 0.0), (4, 2, 64, 32, [300], 24, 0.07), (8, 8, 64, 16, [1000], 0, 0.3),
                                                     (32, 8, 128, 8, [513], 128, 0.0), (2, 1, 64, 8, [8 + 3 * i for i in range(64)], 0, 0.0),
                                                     (2, 1, 128, 8, [0, 9] + [40] * 60 + [600, 0], 8, 0.05)])
def test_one_scoring_launch_strides_scale_and_batch(sweep_mod, oracle, Hq, G, d, w, lens, pad, scale, dtype, causal):
    _check_scores(sweep_mod, oracle, Hq, G, d, w, dtype, causal, lens, pad, scale)


# more than 128 rows of 128 components in short key chunks (64 to 416 keys): sequences around the 32-key tiles and the two or three
# of a whole chunk; rows that fill the four waves, that leave one of them idle, that leave part of a block; strides; the rerun
# with the running maximum
@pytest.mark.parametrize("Hq,G,w,lens,pad", [(4, 1, 64, [31, 33, 1, 64, 95, 97, 129, 2049], 0), (8, 8, 130, [33000], 0),
                                             (6, 2, 64, [40000, 70, 1217], 8), (12, 2, 32, [20001, 9000], 0), (40, 1, 8, [33333], 0),
                                             (8, 1, 64, [30000], 0)])
@pytest.mark.parametrize("causal", [False, True])
@pytest.mark.parametrize("late", [0.0, 0.4])
def test_wide_scoring_kernels(sweep_mod, oracle, Hq, G, w, lens, pad, causal, late):
    if causal:
        lens = [n for n in lens if n >= w]
    _check_scores(sweep_mod, oracle, Hq, G, 128, w, torch.bfloat16, causal, lens, pad=pad, two_pass=True, late=late)


# ... and in long ones: the pipelined loop's first and last tiles, its runs of two and the half of one, the tiles requested ahead
# (three), the sums parked (eight), what it leaves to the plain loop (helpers.LONG_CHUNKS; the host tests hold the plan to it)
@pytest.mark.parametrize("Hq,G,w,lens,pad", LONG_CHUNKS)
@pytest.mark.parametrize("causal", [False, True])
@pytest.mark.parametrize("late", [0.0, 0.4])
def test_scoring_in_long_key_chunks(sweep_mod, oracle, Hq, G, w, lens, pad, causal, late):
    _check_scores(sweep_mod, oracle, Hq, G, 128, w, torch.bfloat16, causal, lens, pad=pad, two_pass=True, late=late)


def _select(B, scores, lens, ks, tail):
    total, cu = sum(lens), np.concatenate([[0], np.cumsum(lens)]).tolist()
    ws = torch.full((max(B.structkv_workspace_bytes(None, len(lens), total), 256),), 0xA5, dtype=torch.uint8, device="cuda")
    out = torch.full((sum(ks) + tail * len(ks) + 1,), -7, dtype=torch.int32, device="cuda")
    B.structkv_select_topk(scores, cu, ks, tail, out, ws)
    got = out.cpu().numpy()
    assert got[-1] == -7
    return got[:-1]


# the edges of the three forms (8192 and 262144 searched scores), of their 1024-score workgroups and of the candidate
# lists (2048 per sequence, 256 in a near bin); scores: spread, crowded to a few and to a few tenths of a per cent, nearly equal (a crowd around
# a power of two), all equal, alternating between two values a power apart (a sample that misses the threshold's range),
# zeros with as many others as are kept, a crowd of a few different keys, a crowd far below what a sample shows (its sub-bin's
# keys are neither few nor equal), negative
@pytest.mark.parametrize("lens,tail", [([1], 0), ([63, 64, 65], 3), ([1025], 1), ([8192 + 8], 8), ([8193 + 8], 8), ([9216, 5, 0], 0),
                                       ([17000, 20000], 32), ([262144 + 7], 7), ([262145 + 7, 300], 7), ([33000] * 17, 64)])
@pytest.mark.parametrize("kind", ["spread", "crowd", "dense", "close", "equal", "two", "cliff", "steps", "ledge", "negative"])
def test_selection_forms(B, oracle, lens, tail, kind):
    total = sum(lens)
    x = _randn(total, dtype=torch.float32, seed=3)
    u = _randn(total, dtype=torch.float32, seed=4)
    scores = {"spread": torch.exp(4.0 * x), "crowd": 1.3 + 0.03 * x, "dense": 1.3 + 0.002 * x, "close": 1.0 + 1e-5 * x,
              "equal": torch.full_like(x, 0.25), "two": torch.where(x > 2.5, 1e20, 1e-20) * (1.0 + 0.1 * x.abs()),
              "cliff": torch.where(u > 0.8416, 1.0 + 0.02 * x, torch.zeros_like(x)),
              "ledge": torch.where(u > 0.8779, 1.0 + 0.02 * x, 1e-20 * (1.0 + 0.1 * x.abs())),
              "steps": torch.where(u > 2.0, 1.0 + x.abs(), 1e-4 * (1.0 + 2e-7 * torch.floor(x))), "negative": -torch.exp(x)}[kind].contiguous()
    for frac in (0.0, 0.003, 0.2, 1.0):
        ks = [int(frac * max(n - tail, 0)) if n >= tail else 0 for n in lens]
        t = min([tail] + lens)
        ref = oracle.select_topk(scores.cpu().numpy(), lens, ks, t)
        assert np.array_equal(_select(B, scores, lens, ks, t), np.concatenate(ref)), (kind, frac)


# the time of a selection must not depend on how close its scores lie: digit passes over the scores took at most 1.3 times
# as long for any of these as for spread scores, a placement that reads all scores again in every workgroup 15 to 28 times
@pytest.mark.parametrize("n", [131072, 262144])
def test_time_of_crowded_selections(B, n):
    x, u = _randn(n, dtype=torch.float32, seed=1), _randn(n, dtype=torch.float32, seed=2)
    kinds = {"spread": torch.exp(0.5 * x), "few per cent": 1.3 + 0.03 * x, "per cent": 1.3 + 0.01 * x, "per mille": 1.3 + 0.003 * x,
             "nearly equal": 1.0 + 1e-5 * x, "equal": torch.full_like(x, 0.25),
             "cliff": torch.where(u > 0.8416, 1.0 + 0.02 * x, torch.zeros_like(x)),
             "zeros": torch.where(u > 3.0, 1.0 + 0.02 * x, torch.zeros_like(x)), "two values": torch.where(u > 0.9, 4.0, 1.0)}
    ws = torch.empty(B.structkv_workspace_bytes(None, 1, n), dtype=torch.uint8, device="cuda")
    times = {}
    for kind, scores in kinds.items():
        for frac in (0.1, 0.2):
            k = int(frac * n)
            out = torch.empty(k, dtype=torch.int32, device="cuda")
            best = float("inf")
            for rep in range(6):
                start, stop = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
                start.record()
                for _ in range(10):
                    B.structkv_select_topk(scores, [0, n], [k], 0, out, ws)
                stop.record()
                stop.synchronize()
                best = min(best, start.elapsed_time(stop))
            times[kind, frac] = best
    for kind, frac in times:
        assert times[kind, frac] <= 3.0 * times["spread", frac], (kind, frac, times)


# a layer step's selection on the in-degrees it has just formed: all in-degrees equal (every score a candidate), budgets
# of one and of everything, sequences on both sides of the short form's limit
@pytest.mark.parametrize("lens,ks", [([20000], [700]), ([20000], [1]), ([9000, 40, 100], [8968, 8, 0]), ([8192 + 32, 50], [8192, 1]),
                                     ([300000], [1000])])
@pytest.mark.parametrize("zero", [False, True])
def test_layer_step_selection_forms(sweep_mod, oracle, lens, ks, zero):
    w = 32
    sw = sweep_mod.LayerSweep(4, 2, 64, w, torch.bfloat16, lens, ks)
    q = _randn(len(lens), 4, w, 64, dtype=torch.bfloat16, seed=4) * (0.0 if zero else 3.0)
    k, v = (_randn(2, sum(lens), 64, dtype=torch.bfloat16, seed=s) for s in (5, 6))
    sw.layer(q, k, v)
    idx = sw.idx_kv.cpu().numpy()[:sw.rows]
    ref = np.concatenate(oracle.select_topk(sw.indeg.cpu().numpy(), lens, ks, w))
    assert np.array_equal(idx, ref)


def _check_pivot(sweep_mod, oracle, Hq, G, d, w, lens, causal):
    total = sum(lens)
    sw = sweep_mod.LayerSweep(Hq, G, d, w, torch.bfloat16, lens, [0] * len(lens), causal=causal)
    q = _randn(len(lens), Hq, w, d, dtype=torch.bfloat16, seed=7)
    k = _randn(G, total, d, dtype=torch.bfloat16, seed=8)
    rho, var = sw.score_pivot(q, k)
    D, ent, _, probs = oracle.score_layer(to_oracle_array(q), to_oracle_array(k), Hq, G, d, w, lens, causal=causal, want_probs=True)
    rho_ref, var_ref = oracle.pivot_metrics(probs, 0.1)
    assert_close_floor(sw.indeg.cpu().numpy(), D, 1e-3, "indeg")
    assert_entropy(sw.entropy.cpu().numpy()[:len(lens)], ent, 1e-3)
    assert np.all(np.abs(rho.cpu().numpy()[:len(lens)] - rho_ref) <= 1e-3 * rho_ref)
    # a variance is a sum of squared differences from 1/n: relative to their squares as in the other parity tests
    assert np.all(np.abs(var.cpu().numpy()[:len(lens)] - var_ref) <= 2e-3 * var_ref + 1e-4 / np.array(lens, dtype=np.float64) ** 2)


# per-head planes with several heads per 32-row block (windows of 8 and 16): one- and four-wave workgroups, one and two
# row blocks per wave, groups whose last wave or block is partly empty, chunks of less than the three direct tiles, sequences of a few tokens
# (from four on the metrics come from the planes)
@pytest.mark.parametrize("Hq,G,d,w,lens", [(32, 8, 128, 8, [700, 33, 1500]), (4, 4, 64, 8, [40, 300]), (16, 2, 128, 8, [2100]),
                                           (24, 2, 128, 8, [1000]), (34, 2, 64, 8, [1300, 65]), (32, 8, 128, 16, [999]),
                                           (5, 1, 128, 16, [513, 97]), (3, 1, 64, 16, [64]), (18, 2, 128, 16, [1111]),
                                           (10, 2, 128, 32, [1400]), (4, 2, 128, 32, [3, 4, 5, 6, 7]), (24, 2, 128, 8, [4, 5, 9])])
@pytest.mark.parametrize("causal", [False, True])
def test_pivot_metrics_of_short_windows(sweep_mod, oracle, Hq, G, d, w, lens, causal):
    if causal:
        lens = [max(n, w) for n in lens]
    _check_pivot(sweep_mod, oracle, Hq, G, d, w, lens, causal)


# ... in long key chunks of more than 128 rows: the pipelined loop with planes, what it collects in LDS and what it writes directly
# (helpers.LONG_CHUNKS_PIVOT; the host tests hold the plan to it)
@pytest.mark.parametrize("Hq,G,w,n", LONG_CHUNKS_PIVOT)
@pytest.mark.parametrize("causal", [False, True])
def test_pivot_metrics_in_long_key_chunks(sweep_mod, oracle, Hq, G, w, n, causal):
    _check_pivot(sweep_mod, oracle, Hq, G, 128, w, [n], causal)


# the top-k mass of the per-head rows: shares of 4096 scores and their remainders; scores within a few per cent (the fine bins),
# over many octaves (a threshold among the quarter octaves), and all equal (one bin holds the row: as many candidates as keys, around
# what eight and sixteen waves hold two a thread, and more than the registers take, 32768).  sharp scales the queries.
@pytest.mark.parametrize("n", [64, 1024, 1025, 2048, 2049, 4095, 4096, 4097, 9000, 16385, 32768, 32769, 40000])
@pytest.mark.parametrize("sharp", [0.0, 0.2, 1.0, 12.0])
def test_pivot_rows(sweep_mod, oracle, n, sharp):
    Hq, G, d, w = 4, 2, 64, 32
    sw = sweep_mod.LayerSweep(Hq, G, d, w, torch.bfloat16, [n], [0])
    q = (_randn(1, Hq, w, d, dtype=torch.float32, seed=11) * sharp).to(torch.bfloat16)
    k = _randn(G, n, d, dtype=torch.bfloat16, seed=12)
    D, ent, _, probs = oracle.score_layer(to_oracle_array(q), to_oracle_array(k), Hq, G, d, w, [n], want_probs=True)
    rho_ref, var_ref = oracle.pivot_metrics(probs, 0.1)
    for _ in range(2):   # a call leaves nothing behind that changes the next
        sw.indeg.fill_(-1.0)
        rho, var = sw.score_pivot(q, k)
        assert_close_floor(sw.indeg.cpu().numpy(), D, 1e-3, "indeg")
        assert_entropy(sw.entropy.cpu().numpy()[:1], ent, 1e-3)
        assert np.all(np.abs(rho.cpu().numpy()[:1] - rho_ref) <= 1e-3 * rho_ref)
        assert np.all(np.abs(var.cpu().numpy()[:1] - var_ref) <= 2e-3 * var_ref + 1e-4 / n ** 2)


# short inputs: key chunks of 64 .. 256 keys (two to eight tiles), one- and four-wave workgroups
@pytest.mark.parametrize("Hq,G,w", [(8, 2, 8), (4, 2, 32), (8, 2, 32), (8, 2, 64)])
@pytest.mark.parametrize("lens", [[64], [65, 1, 0, 200], [5000], [17000, 31]])
def test_short_key_chunks(sweep_mod, oracle, Hq, G, w, lens):
    _check_scores(sweep_mod, oracle, Hq, G, 128, w, torch.bfloat16, False, lens, two_pass=True)


# short sequences in one scoring launch: edges of the 16-key tiles, of the two, four and eight tiles per wave (512, 1024,
# 2048 keys) and of the path itself (1024 fp32 / 1792 or 2048 bf16 keys, 64 column-sum planes), rows around the 16- and 32-row
# blocks, one and two row blocks per workgroup, empty sequences; then the layer step, whose selection forms the in-degrees itself, against the separate calls
@pytest.mark.parametrize("Hq,G,d,w", [(1, 1, 64, 1), (3, 1, 128, 5), (8, 8, 64, 32), (32, 8, 128, 8), (4, 2, 64, 17), (16, 2, 128, 64),
                                      (32, 8, 64, 64)])
@pytest.mark.parametrize("lens", [[1], [15, 0, 17], [255, 256, 257], [512, 513], [1024], [1025, 33], [1281, 1536], [1792], [1793],
                                  [2048], [2049, 5]])
@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("causal", [False, True])
def test_short_sequences_in_one_scoring_launch(sweep_mod, oracle, Hq, G, d, w, lens, dtype, causal):
    if causal:
        lens = [max(n, w) if n else 0 for n in lens]
    _check_scores(sweep_mod, oracle, Hq, G, d, w, dtype, causal, lens)
    lens = [max(n, w) for n in lens]
    ks = [(n - w) // 3 for n in lens]
    q = _randn(len(lens), Hq, w, d, dtype=dtype, seed=9)
    k, v = (_randn(G, sum(lens), d, dtype=dtype, seed=s) for s in (10, 11))
    sweeps = [sweep_mod.LayerSweep(Hq, G, d, w, dtype, lens, ks, causal=causal) for _ in range(2)]
    for _ in range(2):   # (the second layer updates a centrality that is not zero)
        sweeps[0].layer(q, k, v)
        sweeps[1].layer_separate_calls(q, k, v)
    for name in ("indeg", "centrality", "entropy", "entropy_per_head", "idx_kv", "k_cache", "v_cache"):
        assert torch.equal(getattr(sweeps[0], name), getattr(sweeps[1], name)), name


# ... and the same plan with a workspace that only the two-pass plan fits
@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
def test_short_sequences_with_a_smaller_workspace(B, oracle, dtype):
    Hq, G, d, w, n = 16, 2, 64, 64, 900
    code = B.STRUCTKV_DTYPE_F32 if dtype == torch.float32 else B.STRUCTKV_DTYPE_BF16
    shape = B.make_shape(Hq, G, d, w, code)
    need = B.structkv_workspace_bytes(shape, 1, n)
    q, k = _randn(1, Hq, w, d, dtype=dtype, seed=12), _randn(G, n, d, dtype=dtype, seed=13)
    D, ent, ent_h, _ = oracle.score_layer(to_oracle_array(q), to_oracle_array(k), Hq, G, d, w, [n])
    tol = 1e-5 if dtype == torch.float32 else 1e-3
    refused = 0
    for nbytes in range(need, 0, -max(need // 16 // 256 * 256, 256)):
        out, e, eh = torch.zeros(n, device="cuda"), torch.zeros(1, device="cuda"), torch.zeros(1, Hq, device="cuda")
        ws = torch.full((nbytes,), 0xA5, dtype=torch.uint8, device="cuda")
        try:
            B.structkv_score_layer(shape, q, k, [0, n], out, e, eh, ws)
        except B.StructKVError as err:
            assert err.status == B.STRUCTKV_ERR_WORKSPACE and nbytes < need
            refused += 1
            continue
        assert not refused   # (a larger one was accepted)
        assert_close_floor(out.cpu().numpy(), D, tol, "indeg")
        assert_entropy(e.cpu().numpy(), ent, tol)


# the size of the workspace, from the reported one on, does not show in the results
@pytest.mark.parametrize("dtype,lens", [(torch.float32, [900]), (torch.bfloat16, [900]), (torch.bfloat16, [700, 33, 1500, 64]),
                                        (torch.bfloat16, [3000, 5])])
def test_results_do_not_depend_on_a_larger_workspace(B, dtype, lens):
    Hq, G, d, w = 16, 2, 64, 32
    shape = B.make_shape(Hq, G, d, w, B.STRUCTKV_DTYPE_F32 if dtype == torch.float32 else B.STRUCTKV_DTYPE_BF16)
    need = B.structkv_workspace_bytes(shape, len(lens), sum(lens))
    q, k = _randn(len(lens), Hq, w, d, dtype=dtype, seed=12), _randn(G, sum(lens), d, dtype=dtype, seed=13)
    cu = np.concatenate([[0], np.cumsum(lens)]).tolist()
    outs = []
    for nbytes in (need, need + 256, 4 * need):
        out, e, eh = torch.zeros(sum(lens), device="cuda"), torch.zeros(len(lens), device="cuda"), torch.zeros(len(lens), Hq, device="cuda")
        B.structkv_score_layer(shape, q, k, cu, out, e, eh, torch.full((nbytes,), 0xA5, dtype=torch.uint8, device="cuda"))
        outs.append((out, e, eh))
    for other in outs[1:]:
        assert all(torch.equal(a, b) for a, b in zip(outs[0], other))


# inputs that are not finite: a NaN key makes its whole sequence NaN (in the masked tiles too), a NaN query row reaches
# the keys that it sees and no others; the sequences beside it are untouched
@pytest.mark.parametrize("dtype,w,lens", [(torch.float32, 32, [1500, 40]), (torch.float32, 8, [900, 300]), (torch.bfloat16, 8, [3000, 90]),
                                          (torch.bfloat16, 64, [5000, 64]), (torch.bfloat16, 8, [700, 33]), (torch.bfloat16, 64, [1000, 65]),
                                          (torch.bfloat16, 64, [50979, 65])])
@pytest.mark.parametrize("causal", [False, True])
@pytest.mark.parametrize("value", [float("nan"), float("inf")])
def test_inputs_that_are_not_finite(sweep_mod, oracle, dtype, w, lens, causal, value):
    Hq, G, d = 8, 2, 128
    q, k = _randn(2, Hq, w, d, dtype=dtype, seed=14), _randn(G, sum(lens), d, dtype=dtype, seed=15)
    tol = 1e-5 if dtype == torch.float32 else 1e-3
    D, ent, _, _ = oracle.score_layer(to_oracle_array(q), to_oracle_array(k), Hq, G, d, w, lens, causal=causal)
    n = lens[0]
    sw = sweep_mod.LayerSweep(Hq, G, d, w, dtype, lens, [0, 0], causal=causal)
    for key in (0, n // 2, n - w, n - w + 3, n - 1):
        bad = k.clone()
        bad[1, key] = value   # (an infinite key: logits of both signs, or NaN)
        sw.score(q, bad)
        got, e = sw.indeg.cpu().numpy(), sw.entropy.cpu().numpy()
        assert np.isnan(got[:n]).all() and np.isnan(e[0]), key   # (the window's last row sees every key)
        assert_close_floor(got[n:], D[n:], tol, "the other sequence")
        assert_entropy(e[1:2], ent[1:2], tol)
    for row in (0, 3, w - 1):
        bad = q.clone()
        bad[0, 5, row] = float("nan")
        sw.score(bad, k)
        got = sw.indeg.cpu().numpy()
        seen = n - w + row + 1 if causal else n
        assert np.isnan(got[:seen]).all() and not np.isnan(got[seen:]).any(), row
        assert_close_floor(got[n:], D[n:], tol, "the other sequence")
