"""Importance of prompts of up to 2048 tokens in one pass, at the edges of its blocks, waves and shares, and
where a row block has to be formed again with exact maxima, against the fp64 oracle."""
import numpy as np
import pytest
import torch

import oracle
import paper_2608_15592_amd as estp
from synth import inputs as I
from tests._util import dev, host

pytestmark = pytest.mark.gpu

U = 2.0 ** -24


def _qk(lengths, L, Hq, Hkv, dh, seed, qscale=1.0):
    g = np.random.default_rng(seed)
    n = sum(lengths)
    Q = I.f32_to_bf16_bits(qscale * g.standard_normal((L, n, Hq, dh)).astype(np.float32))
    K = I.f32_to_bf16_bits(g.standard_normal((L, n, Hkv, dh)).astype(np.float32))
    return Q, K, I.cu_seqlens_from_lengths(lengths)


def _rtol(Q, K, scale, n_max):
    """Relative bound on S: a score is within gamma_(dh + 1) of the sum of its products' sizes (at most
    |q||k|), a probability within exp(2 delta) - 1 of its value, and sums of positive terms add an ulp a term."""
    q = np.linalg.norm(oracle.widen(Q), axis=-1).max()
    k = np.linalg.norm(oracle.widen(K), axis=-1).max()
    delta = (Q.shape[-1] + 1) * U * scale * q * k
    return np.expm1(2 * delta) + (n_max + 64) * U


CASES = [
    # lengths, L, Hq, Hkv, dh
    ([1], 1, 4, 1, 128),
    ([31, 32, 33], 1, 4, 2, 32),
    ([255, 256, 257], 2, 2, 2, 64),       # eight row blocks and one past, a head of its own per KV head
    ([1024], 1, 4, 1, 128),               # the most of four waves
    ([1025], 1, 3, 1, 64),                # the least of eight
    ([2048], 1, 2, 1, 128),               # the most of eight
    ([2048, 1500, 1170], 1, 1, 1, 32),
    ([40, 900, 3, 64, 129, 512, 7], 1, 6, 2, 128),  # a small ragged batch
]


@pytest.mark.parametrize("lengths,L,Hq,Hkv,dh", CASES, ids=["-".join(map(str, c[0])) + f"-dh{c[4]}" for c in CASES])
def test_onepass_parity(lengths, L, Hq, Hkv, dh):
    Q, K, cu = _qk(lengths, L, Hq, Hkv, dh, 3)
    Qd, Kd, cud = dev(Q), dev(K), dev(cu)
    rtol = _rtol(Q, K, dh ** -0.5, max(lengths))
    S = estp.attn_importance(Qd, Kd, cud, max(lengths))
    ref = oracle.attn_importance(Q, K, cu)
    print(f"max rel |dS| / bound = {(np.abs(host(S) - ref) / ref / rtol).max():.3g}")
    assert np.all(np.abs(host(S) - ref) <= rtol * ref)
    assert torch.equal(S, estp.attn_importance(Qd, Kd, cud, max(lengths)))
    # the general kernels on the same call (a bound on the lengths past the one pass)
    if sum(lengths) >= 2049:
        S2 = estp.attn_importance(Qd, Kd, cud, 2049)
        assert np.all(np.abs(host(S2) - host(S)) <= 2 * rtol * ref)
    # layer weights and the diagonal left out; the first token of a one-token prompt then gets exactly 0
    w = [0.5 + l for l in range(L)]
    S = host(estp.attn_importance_ex(Qd, Kd, cud, max(lengths), layer_weights=w, exclude_self=True))
    ref = oracle.attn_importance(Q, K, cu, layer_weights=w, exclude_self=True)
    assert np.all(np.abs(S - ref) <= rtol * np.abs(ref) + 2.0 ** -126)


@pytest.mark.parametrize("tag", ["sharp", "all-low", "some-rows"])
def test_onepass_sums_out_of_range(tag):
    lengths, dh = [300, 70], 64
    Q, K, cu = _qk(lengths, 1, 4, 2, dh, 4, qscale=40.0 if tag != "all-low" else 1.0)
    if tag == "all-low":  # every score near -250 nats: the sums underflow
        g = np.random.default_rng(5)
        v = np.sign(g.standard_normal(dh)).astype(np.float32)
        Q = I.f32_to_bf16_bits(6 * np.broadcast_to(v, Q.shape).astype(np.float32) + I.bf16_bits_to_f32(Q) * 0.1)
        K = I.f32_to_bf16_bits(-6 * np.broadcast_to(v, K.shape).astype(np.float32) + I.bf16_bits_to_f32(K) * 0.1)
    elif tag == "some-rows":
        q = I.bf16_bits_to_f32(Q)
        q[:, np.arange(q.shape[1]) % 7 != 0] /= 40.0
        Q = I.f32_to_bf16_bits(q)
    S = host(estp.attn_importance(dev(Q), dev(K), dev(cu), max(lengths)))
    ref = oracle.attn_importance(Q, K, cu)
    rtol = _rtol(Q, K, dh ** -0.5, max(lengths))
    print(f"{tag}: bound {rtol:.2e}, max rel |dS| / bound = {(np.abs(S - ref) / ref / rtol).max():.3g}")
    assert np.all(np.abs(S - ref) <= rtol * ref + 2.0 ** -126)


def test_onepass_not_a_number_stays_in_its_rows():
    # a query that is not a number reaches the keys up to its own token, as in the two-pass kernels
    lengths, dh = [200], 64
    Q, K, cu = _qk(lengths, 1, 2, 1, dh, 6)
    q = I.bf16_bits_to_f32(Q)
    q[0, 70, 1] = np.nan
    S = host(estp.attn_importance(dev(I.f32_to_bf16_bits(q)), dev(K), dev(cu), 200))
    assert np.all(np.isnan(S[:71]))
    assert np.all(np.isfinite(S[71:]))


def _walk(lengths, L, Hq, Hkv):
    """Row blocks that one workgroup of the one-pass kernel takes at least, over its heads, in the longest prompt: the
    shares of a call reach four (eight waves) or eight workgroups per compute unit and no further."""
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    G, nrb = Hq // Hkv, (max(lengths) + 31) // 32
    want = (4 if max(lengths) > 1024 else 8) * cus
    units = len(lengths) * L * Hkv
    rsplit, hsplit = max(1, min(8, G * nrb // 16)), 1
    while rsplit < min(8, nrb) and units * rsplit < want:
        rsplit += 1
    while hsplit < G and (G % hsplit or units * rsplit * hsplit < want):
        hsplit += 1
    if units * rsplit * hsplit < want:
        rsplit = min(nrb, -(-want // (units * hsplit)))
    return nrb // rsplit * (G // hsplit)


# workgroups of four and of eight waves that walk several row blocks of several heads
WALK_CASES = [([512] * 16, 1, 32, 8, 128), ([1057] * 4, 1, 32, 8, 32), ([330, 500, 441] * 11, 1, 8, 4, 64)]


@pytest.mark.parametrize("rows", ["first-low", "first-high", "middle", "scattered", "all", "spread"])
@pytest.mark.parametrize("lengths,L,Hq,Hkv,dh", WALK_CASES, ids=["w4-dh128", "w8-dh32", "w4-dh64-ragged"])
def test_onepass_sums_out_of_range_between_others(lengths, L, Hq, Hkv, dh, rows):
    # row blocks formed again between ordinary ones: the queries of the next block or head arrive meanwhile
    assert _walk(lengths, L, Hq, Hkv) >= 2
    g = np.random.default_rng(7)
    n = sum(lengths)
    at = np.concatenate([np.arange(N) for N in lengths])  # position in the prompt
    far = {"first-low": at < 3, "first-high": at < 3, "middle": (at >= 200) & (at < 210), "scattered": at % 37 == 0,
           "all": np.ones(n, bool), "spread": np.ones(n, bool)}[rows]
    v = np.sign(g.standard_normal(dh)).astype(np.float32)
    c = 90.0 / np.sqrt(dh) * (-1.0 if rows in ("first-low", "all") else 1.0)  # scores near -90 or 90 nats
    K = I.f32_to_bf16_bits((v + 0.1 * g.standard_normal((L, n, Hkv, dh))).astype(np.float32))
    q = g.standard_normal((L, n, Hq, dh))
    q -= (q @ v)[..., None] * v / dh
    q[:, far] = 0.5 * q[:, far] + c * v
    if rows == "spread":  # scores of 40 nats' standard deviation: the waves' maxima lie far apart
        q, K = 40.0 * g.standard_normal((L, n, Hq, dh)), I.f32_to_bf16_bits(g.standard_normal(K.shape).astype(np.float32))
    Q = I.f32_to_bf16_bits(q.astype(np.float32))
    cu = I.cu_seqlens_from_lengths(lengths)
    rtol = _rtol(Q, K, dh ** -0.5, max(lengths))
    Qd, Kd, cud = dev(Q), dev(K), dev(cu)
    S = estp.attn_importance(Qd, Kd, cud, max(lengths))
    ref = oracle.attn_importance(Q, K, cu)
    err = np.abs(host(S) - ref) / (rtol * ref + 2.0 ** -126)
    print(f"{rows}: bound {rtol:.2e}, max |dS| / bound = {err.max():.3g}")
    assert np.all(np.abs(host(S) - ref) <= rtol * ref + 2.0 ** -126)
    assert torch.equal(S, estp.attn_importance(Qd, Kd, cud, max(lengths)))
    X = host(estp.attn_importance_ex(Qd, Kd, cud, max(lengths), exclude_self=True))
    ref = oracle.attn_importance(Q, K, cu, exclude_self=True)
    assert np.all(np.abs(X - ref) <= rtol * ref + 2.0 ** -126)


@pytest.mark.parametrize("rows", ["ordinary", "low"])
@pytest.mark.parametrize("lengths", [[70], [1, 333, 64, 45]], ids=["70", "ragged"])
def test_onepass_infinite_key_feature_gets_no_attention(lengths, rows):
    # a key whose every score is -inf gets exactly 0, also where the last row block has rows past the prompt
    dh = 64
    Q, K, cu = _qk(lengths, 1, 4, 2, dh, 8)
    q, k = I.bf16_bits_to_f32(Q), I.bf16_bits_to_f32(K)
    q[..., 5] = 1.0
    if rows == "low":  # every other score near -95 nats: the rows are formed again
        q[..., 7], k[..., 7] = 32.0, -24.0
    keys = [int(lo) + j for lo, N in zip(cu, lengths) for j in (1, N // 2, N - 1) if N > 1]
    k[:, keys, :, 5] = -np.inf
    Q, K = I.f32_to_bf16_bits(q), I.f32_to_bf16_bits(k)
    S = host(estp.attn_importance(dev(Q), dev(K), dev(cu), max(lengths)))
    ref = oracle.attn_importance(Q, K, cu)
    assert np.all(S[keys] == 0)
    rest = np.setdiff1d(np.arange(sum(lengths)), keys)
    k[..., 5] = 0.0  # the bound of the finite scores
    rtol = _rtol(Q, I.f32_to_bf16_bits(k), dh ** -0.5, max(lengths)) + 8 * U
    assert np.all(np.abs(S[rest] - ref[rest]) <= rtol * ref[rest])
