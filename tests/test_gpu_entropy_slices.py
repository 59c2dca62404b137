"""Vocabulary slices of the entropy call against the fp64 oracle, where the split changes: bf16, the token
tiles past the last whole group of 16 take as many slices as give up to 256 workgroups."""
import numpy as np
import pytest
import torch

import oracle
import paper_2608_15592_amd as estp
from synth import inputs as I
from tests._util import check_vocab_argmax, dev, host, logit_error_bound

# (n_tok, d, V): V in 256-row tiles, tokens in 256-token tiles
CASES = [
    (1, 64, 16400),      # one token
    (256, 96, 70000),    # 32-deep stages
    (257, 64, 16400),
    (2304, 64, 8200),    # 9 tiles: two column groups of 5 and 4, 28 slices
    (3840, 32, 4353),    # 15 tiles, 17 slices, odd multiple of 32
    (4096, 64, 4353),    # one whole group, nothing past it
    (4097, 64, 8200),    # one whole group and one token past it
    (4700, 64, 4097),    # 17 vocabulary tiles, the last one row; three tiles past the group
    (300, 64, 4096),     # 16 vocabulary tiles: never more than 16 slices
]


CASES_F32 = [
    (1, 8, 1),
    (63, 40, 65),        # depth ends inside a step
    (65, 72, 129),       # one token and one word past a tile
    (129, 64, 16500),
    (4097, 32, 300),     # few vocabulary tiles
]


def _check(X, W, n, V):
    am = torch.full((n,), -7, dtype=torch.int32, device="cuda")
    Xd, Wd = dev(X), dev(W)
    H = estp.token_entropy(Xd, Wd, vocab_argmax=am)
    rows = np.unique(np.concatenate([np.arange(min(n, 40)), np.arange(max(0, n - 300), n), np.arange(0, n, 61)]))
    ref = oracle.token_entropy(X[rows], W)
    # H moves by at most sum_v p_v |z_v - E z| |dz| <= (ln V + max z - min z) max|dz| with logit errors
    # below half logit_error_bound; the exp2, log2 and sums of positive terms add a few hundred ulp of H,
    # and of 1 where H itself is small
    z = oracle.widen(X[rows]) @ oracle.widen(W).T
    bound = ((np.log(V) + z.max(axis=1) - z.min(axis=1)) * logit_error_bound(X, W, rows) / 2
             + 300 * 2.0 ** -24 * np.maximum(ref, 1.0))
    err = np.abs(host(H)[rows] - ref)
    print(f"max |dH| / bound = {(err / bound).max():.3g}")
    assert np.all(err <= bound)
    check_vocab_argmax(host(am)[rows], X, W, rows)
    # without the mode, and on the library's own scratch: the same bits
    assert torch.equal(estp.token_entropy(Xd, Wd), H)
    assert torch.equal(estp.token_entropy_noalloc(Xd, Wd, torch.empty_like(H)), H)


def _inputs(n, d, V):
    g = np.random.default_rng(n + V)
    X = g.standard_normal((n, d)).astype(np.float32)
    return X / np.sqrt((X * X).mean(axis=1, keepdims=True)), g.standard_normal((V, d)).astype(np.float32) * 0.3


@pytest.mark.gpu
@pytest.mark.parametrize("n,d,V", CASES, ids=["x".join(map(str, c)) for c in CASES])
def test_entropy_slices(n, d, V):
    X, W = _inputs(n, d, V)
    _check(I.f32_to_bf16_bits(X), I.f32_to_bf16_bits(W), n, V)


@pytest.mark.gpu
@pytest.mark.parametrize("n,d,V", CASES_F32, ids=["x".join(map(str, c)) for c in CASES_F32])
def test_entropy_slices_f32(n, d, V):
    X, W = _inputs(n, d, V)
    _check(X, W, n, V)


@pytest.mark.gpu
@pytest.mark.parametrize("d,V", [(64, 33000), (192, 4097), (128, 40000), (64, 300)])
def test_few_tokens_change_no_bit(d, V):
    # a call of up to 2048 tokens spreads the same arithmetic over more workgroups: its rows of a call of
    # one whole group of token tiles, bit for bit, with vocabularies of a ragged last tile, of tiles that
    # do not fill the last product of a slice, and of fewer tiles than slices; at block edges of the tokens
    X, W = _inputs(4096, d, V)
    W[V // 2:] *= 40.0  # later tiles far above the running reference: folded exactly
    Xd, Wd = dev(I.f32_to_bf16_bits(X)), dev(I.f32_to_bf16_bits(W))
    am = torch.empty(4096, dtype=torch.int32, device="cuda")
    H = estp.token_entropy(Xd, Wd, vocab_argmax=am)
    for n in (1, 63, 64, 65, 200, 719, 2048):
        x = Xd[:n].contiguous()
        a = torch.full((n,), -7, dtype=torch.int32, device="cuda")
        assert torch.equal(estp.token_entropy(x, Wd, vocab_argmax=a), H[:n])
        assert torch.equal(a, am[:n])
        assert torch.equal(estp.token_entropy(x, Wd), H[:n])


def test_entropy_workspace_grows_with_tokens():
    # a workspace sized for more tokens serves fewer, and the no-allocation limit holds for every vocabulary
    for V in (1, 300, 4096, 4097, 33000, 151936):
        sizes = [estp.token_entropy_workspace_size(n, 64, V) for n in
                 (1, 2, 255, 256, 257, 3840, 4096, 4097, 60000, 98303, 98304, 98305, 102400, 104856)]
        assert sizes == sorted(sizes)
        assert sizes[-1] <= estp._lib.ESTP_NOALLOC_SCRATCH_BYTES
