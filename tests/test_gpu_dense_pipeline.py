"""The software-pipelined dense groups (256 queries at head_dim 128, else 128;
rings of four or two key-value tiles): the shortest group, lengths around the
ring's and the unrolled loop's wrap, and repeated passes, against the oracle."""

import numpy as np
import pytest
import torch

from oracle import wise_oracle as O
from parity_util import ACC_TOL, assert_attn, assert_lse, f64

pytestmark = pytest.mark.gpu


# Waves with 1 to 20 tiles, so every remainder of the unrolled loop and every
# state of the rings occurs; d 128 lengths that 256 does not divide run 4-wave
# groups.
@pytest.mark.parametrize("n,B,heads,kv_heads,d", [
    (256, 64, 1, 1, 128), (512, 16, 2, 1, 128), (768, 128, 3, 3, 128), (1280, 32, 4, 2, 128),
    (128, 16, 1, 1, 128), (640, 128, 2, 2, 128), (128, 64, 2, 1, 64), (384, 32, 3, 3, 64),
    (1152, 128, 2, 1, 64), (128, 32, 1, 1, 96), (256, 128, 2, 2, 96), (896, 16, 2, 1, 96)])
def test_pipelined_dense_group(gpu_lib, n, B, heads, kv_heads, d):
    w = gpu_lib
    g = torch.Generator().manual_seed(n + B + d)
    q = (torch.randn((1, heads, n, d), generator=g) * 2).to(torch.bfloat16)
    k, v = (torch.randn((1, kv_heads, n, d), generator=g).to(torch.bfloat16) for _ in range(2))
    s = w.make_shape(1, heads, n, d, B, kv_heads=kv_heads)
    qd, kd, vd, ws = q.cuda(), k.cuda(), v.cuda(), w.mass_workspace(s)
    first = None
    for _ in range(4):     # the same bits every time: no pass reads a tile before it landed
        o, lse = torch.empty_like(qd), torch.empty((1, heads, n), device="cuda")
        acc = torch.zeros((1, heads, n // B, n // B), device="cuda")
        plain = torch.empty_like(qd)
        w.wise_dense_attn_accum(s, qd, kd, vd, o, lse, acc, ws)
        w.wise_dense_attn_accum(s, qd, kd, vd, plain, None, None)
        torch.cuda.synchronize()
        if first is None:
            first = (o, lse, acc, plain)
        assert all(torch.equal(a, b) for a, b in zip(first, (o, lse, acc, plain)))
    qe, ke, ve = f64(q), O.expand_kv(f64(k), heads), O.expand_kv(f64(v), heads)
    o_ref, l_ref = O.dense_attention(qe, ke, ve)
    assert_attn(first[0], o_ref, f"n={n} B={B} d={d}")
    assert_attn(first[3], o_ref, "without masses")     # its row sums run in another order
    assert_lse(first[1], l_ref)
    assert np.abs(f64(first[2]) - O.block_mass(qe, ke, B)).max() <= ACC_TOL


@pytest.mark.parametrize("n,B,few,many", [(512, 64, 1, 161), (768, 128, 106, 107), (1024, 16, 3, 81), (1280, 32, 64, 65)])
def test_small_grid_gives_the_same_bits(gpu_lib, n, B, few, many):
    """head_dim 128: 320 groups of 256 queries at most run as groups of 128,
    more as they are; a head's outputs do not depend on it."""
    w = gpu_lib
    assert few * n <= 320 * 256 < many * n
    g = torch.Generator(device="cuda").manual_seed(n)
    q, k, v = (torch.randn((1, many, n, 128), generator=g, device="cuda").to(torch.bfloat16) for _ in range(3))
    out = []
    for h in (few, many):
        s = w.make_shape(1, h, n, 128, B)
        qh, kh, vh = (x[:, :h].contiguous() for x in (q, k, v))
        o, lse = torch.empty_like(qh), torch.empty((1, h, n), device="cuda")
        acc = torch.zeros((1, h, n // B, n // B), device="cuda")
        plain = torch.empty_like(qh)
        w.wise_dense_attn_accum(s, qh, kh, vh, o, lse, acc, w.mass_workspace(s))
        w.wise_dense_attn_accum(s, qh, kh, vh, plain, None, None)
        torch.cuda.synchronize()
        out.append([x[:, :few] for x in (o, lse, acc, plain)])
    assert all(torch.equal(a, b) for a, b in zip(*out))
