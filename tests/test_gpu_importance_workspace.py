"""Importance workspaces of another call's size: a short prompt, whose one pass asks for more than a long prompt's two,
runs the two passes in what they need, and nothing less is taken."""
import numpy as np
import pytest
import torch

import oracle
import paper_2608_15592_amd as estp
from paper_2608_15592_amd import _lib
from synth import inputs as I
from tests._util import dev, host

pytestmark = pytest.mark.gpu

S_RTOL = 1e-3  # of the parity tests


def _size(lengths, L, Hq, Hkv, dh):
    n = sum(lengths)
    return _lib.load().estp_attn_importance_workspace_size(n, len(lengths), max(lengths), L, Hq, Hkv, dh,
                                                           _lib.ESTP_BF16)


def _two_pass_size(lengths, L, Hq, Hkv):
    """Row log-sum-exps, column masses and list of live 256-row blocks, 256-byte aligned each."""
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    n, B, G, grid = sum(lengths), len(lengths), Hq // Hkv, len(lengths) * -(-max(lengths) // 256)
    live = min(grid, n // 256 + B)
    blocks = live if 4 * live < 3 * grid else grid
    nsplit = next((d for d in range(1, G) if G % d == 0 and blocks * L * Hkv * d >= 4 * cus), G)
    up = lambda b: -(-b // 256) * 256
    return up(4 * L * Hq * n) + up(4 * L * Hkv * nsplit * n) + up(8 * live)


@pytest.mark.parametrize("n,longer,L,Hq,Hkv,dh", [(1000, 4096, 1, 32, 8, 128), (1030, 2049, 1, 8, 2, 64),
                                                   (300, 3000, 2, 6, 1, 32)])
def test_workspace_of_a_longer_prompt_serves_a_shorter_one(n, longer, L, Hq, Hkv, dh):
    g = np.random.default_rng(n)
    Qh = I.f32_to_bf16_bits(g.standard_normal((L, n, Hq, dh)).astype(np.float32))
    Kh = I.f32_to_bf16_bits(g.standard_normal((L, n, Hkv, dh)).astype(np.float32))
    cu = I.cu_seqlens_from_lengths([n])
    Q, K, cud = dev(Qh), dev(Kh), dev(cu)
    least, told = _two_pass_size([n], L, Hq, Hkv), _size([n], L, Hq, Hkv, dh)
    assert least < told  # the one pass asks for more here
    assert least <= _size([longer], L, Hq, Hkv, dh)
    w = [1.0 + l for l in range(L)]
    ref = oracle.attn_importance(Qh, Kh, cu)
    ref_w = oracle.attn_importance(Qh, Kh, cu, layer_weights=w)
    for nbytes in (told, told - 1, _size([longer], L, Hq, Hkv, dh), least):
        # guard bytes on both sides: neither form writes past the size it was given
        buf = torch.full((nbytes + 512,), 0x5a, dtype=torch.uint8, device="cuda")
        ws = buf[256:256 + nbytes]
        S = host(estp.attn_importance(Q, K, cud, n, workspace=ws))
        assert np.all(np.abs(S - ref) <= S_RTOL * ref), nbytes
        S = host(estp.attn_importance_ex(Q, K, cud, n, layer_weights=w, workspace=ws))
        assert np.all(np.abs(S - ref_w) <= S_RTOL * ref_w), nbytes
        assert bool((buf[:256] == 0x5a).all()) and bool((buf[256 + nbytes:] == 0x5a).all())
    with pytest.raises(estp.EstpError) as e:
        estp.attn_importance(Q, K, cud, n, workspace=torch.empty(least - 1, dtype=torch.uint8, device="cuda"))
    assert e.value.status == _lib.ESTP_ERR_WORKSPACE


@pytest.mark.parametrize("lengths,L,Hq,Hkv,dh", [
    ([1156] * 30, 1, 8, 1, 32),                            # eight waves, mostly without their last key blocks
    ([1187, 593, 890] * 23, 1, 16, 4, 64),
    ([1048, 524, 700, 900, 800, 1000, 600, 868], 1, 48, 8, 128),
    ([1925, 1600, 1790] * 7, 2, 8, 8, 64),
    ([230] * 170, 1, 6, 2, 32),                            # few KV heads: workgroups of a row block or two
    ([335, 280] * 83, 1, 7, 1, 64),
], ids=["8-waves-dh32", "8-waves-dh64", "8-waves-uneven-dh128", "8-waves-uneven-dh64", "shares-dh32", "shares-dh64"])
def test_calls_that_one_pass_would_slow_take_two(lengths, L, Hq, Hkv, dh):
    # measured slower in one pass, by 7 to 36%: they ask for the two passes' arrays and no more.  One prompt alone
    # takes one pass.
    assert _size(lengths, L, Hq, Hkv, dh) == _two_pass_size(lengths, L, Hq, Hkv)
    assert _size(lengths[:1], L, Hq, Hkv, dh) > _two_pass_size(lengths[:1], L, Hq, Hkv)
