"""GPU parity of single kernels at the sizes where they can go wrong: edges of tiles, remainders, the smallest and
largest of their ranges.  Against the fp64 CPU oracle, through the C ABI.

Tolerances: fp32 inputs 1e-5 relative (a dot product of up to 256 fp32 terms is good to a few 1e-7 of its absolute
terms, the exponent to as much absolutely, 2^x to 1 ulp, sums of up to 1e3 of those add 1e-6); bf16 inputs 1e-3, the
bar of the other parity tests.  Selections and copies are exact.
"""
import numpy as np
import pytest
import torch

from helpers import assert_close_floor, assert_entropy, to_oracle_array

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


def _check_scores(sweep_mod, oracle, Hq, G, d, w, dtype, causal, lens, pad=0):
    """Score one layer and compare in-degree and entropies; pad: extra elements between key rows (odd strides)."""
    total = sum(lens)
    sw = sweep_mod.LayerSweep(Hq, G, d, w, dtype, lens, [0] * len(lens), causal=causal)
    q = _randn(len(lens), Hq, w, d, dtype=dtype, seed=1)
    k = _randn(G, total, d + pad, dtype=dtype, seed=2)[:, :, :d]
    sw.indeg.fill_(-7.0)
    sw.score(q, k)
    torch.cuda.synchronize()
    D, ent, ent_h, _ = oracle.score_layer(to_oracle_array(q), to_oracle_array(k), Hq, G, d, w, lens, causal=causal)
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
def test_fp32_matrix_scoring_kernels(sweep_mod, oracle, Hq, G, d, w, lens, pad, dtype, causal):
    if causal:
        lens = [max(n, w) for n in lens]
    _check_scores(sweep_mod, oracle, Hq, G, d, w, dtype, causal, lens, pad)


# causal windows that are no multiple of the 32-row blocks: heads straddle row blocks and waves
@pytest.mark.parametrize("Hq,G,d,w", [(8, 2, 128, 1), (8, 2, 128, 7), (32, 8, 128, 8), (4, 4, 64, 33), (10, 2, 64, 24), (8, 2, 128, 40),
                                      (2, 1, 128, 100)])
def test_causal_windows_on_the_bf16_kernels(sweep_mod, oracle, Hq, G, d, w):
    _check_scores(sweep_mod, oracle, Hq, G, d, w, torch.bfloat16, True, [w, w + 1, 257, 64 + w, 1111])
