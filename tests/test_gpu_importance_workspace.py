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


def _size(n, L, Hq, Hkv, dh):
    return _lib.load().estp_attn_importance_workspace_size(n, 1, n, L, Hq, Hkv, dh, _lib.ESTP_BF16)


def _two_pass_size(n, L, Hq, Hkv):
    """Row log-sum-exps, column masses and block list of one prompt, 256-byte aligned each."""
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    G, blocks = Hq // Hkv, -(-n // 256)
    nsplit = next((d for d in range(1, G) if G % d == 0 and blocks * L * Hkv * d >= 4 * cus), G)
    up = lambda b: -(-b // 256) * 256
    return up(4 * L * Hq * n) + up(4 * L * Hkv * nsplit * n) + up(8 * blocks)


@pytest.mark.parametrize("n,longer,L,Hq,Hkv,dh", [(1000, 4096, 1, 32, 8, 128), (1030, 2049, 1, 8, 2, 64),
                                                   (300, 3000, 2, 6, 1, 32)])
def test_workspace_of_a_longer_prompt_serves_a_shorter_one(n, longer, L, Hq, Hkv, dh):
    g = np.random.default_rng(n)
    Qh = I.f32_to_bf16_bits(g.standard_normal((L, n, Hq, dh)).astype(np.float32))
    Kh = I.f32_to_bf16_bits(g.standard_normal((L, n, Hkv, dh)).astype(np.float32))
    cu = I.cu_seqlens_from_lengths([n])
    Q, K, cud = dev(Qh), dev(Kh), dev(cu)
    least, told = _two_pass_size(n, L, Hq, Hkv), _size(n, L, Hq, Hkv, dh)
    assert least < told  # the one pass asks for more here
    assert least <= _size(longer, L, Hq, Hkv, dh)
    w = [1.0 + l for l in range(L)]
    ref = oracle.attn_importance(Qh, Kh, cu)
    ref_w = oracle.attn_importance(Qh, Kh, cu, layer_weights=w)
    for nbytes in (told, told - 1, _size(longer, L, Hq, Hkv, dh), least):
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
