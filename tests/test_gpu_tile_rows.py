"""64- and 128-key-block rows, whose waves must agree on the tiles that the ids
give, 64 ids at a time: row lengths around that batch, ids to skip at batch
edges, rows with none, odd and even tile counts, against the oracle; and the
kernels for small and for large grids, which give the same bits."""

import numpy as np
import pytest
import torch

from oracle import wise_oracle as O
from parity_util import assert_attn, assert_lse, f64

pytestmark = pytest.mark.gpu


def supports(h, nb, sizes, rng):
    """CSR with ids past the diagonal to skip, and the same without them."""
    rp, ci, clean_rp, clean_ci = [0], [], [0], []
    for r in range(h * nb):
        qb = r % nb
        size = min(qb + 1, int(rng.choice(sizes)))
        row = sorted(rng.choice(qb + 1, size=size, replace=False).tolist())
        past = list(range(qb + 1, min(qb + 1 + int(rng.integers(0, 70)), nb)))
        ci += row + past
        rp.append(len(ci))
        clean_ci += row
        clean_rp.append(len(clean_ci))
    return [np.asarray(x, np.int32) for x in (rp, ci, clean_rp, clean_ci)]


def run(w, q, k, v, B, rp, ci):
    s = w.make_shape(1, q.shape[1], q.shape[2], q.shape[3], B, kv_heads=k.shape[1])
    o, lse = torch.empty_like(q), torch.empty(q.shape[:3], device="cuda")
    w.wise_sparse_attn(s, q, k, v, torch.from_numpy(rp).cuda(), torch.from_numpy(ci).cuda(), None, o, lse)
    torch.cuda.synchronize()
    return o, lse


@pytest.mark.parametrize("B,nb,d,kv_heads", [(64, 132, 64, 1), (64, 132, 96, 2), (64, 132, 128, 2), (128, 72, 64, 2), (128, 72, 96, 1), (128, 72, 128, 1)])
def test_tile_rows_id_batches(gpu_lib, B, nb, d, kv_heads):
    h, n = 2, nb * B
    g = torch.Generator().manual_seed(B + d)
    q = (torch.randn((1, h, n, d), generator=g) * 1.5).to(torch.bfloat16)
    k, v = (torch.randn((1, kv_heads, n, d), generator=g).to(torch.bfloat16) for _ in range(2))
    rp, ci, crp, cci = supports(h, nb, [0, 1, 2, 3, 63, 64, 65, 66, 127, 128, 129], np.random.default_rng(d))
    o, lse = run(gpu_lib, q.cuda(), k.cuda(), v.cuda(), B, rp, ci)
    o_ref, l_ref = O.sparse_attention(f64(q), O.expand_kv(f64(k), h), O.expand_kv(f64(v), h), crp, cci, B)
    assert_attn(o, o_ref, f"B={B} d={d}")
    assert_lse(lse, l_ref)


# Rows (heads x blocks) up to the limit of the kernel with two tiles, one head more (d 96: four groups per CU below
# 2048 rows), and head counts that the XCDs share evenly (40, 32) or not
@pytest.mark.parametrize("d,nb,heads", [(64, 64, (16, 17, 40)), (96, 64, (20, 21, 32, 33)), (128, 64, (12, 13, 40)), (64, 7, (146, 147)), (96, 1, (1280, 1281)),
                                        (128, 2, (384, 385))])
def test_small_and_large_grids_give_the_same_bits(gpu_lib, d, nb, heads):
    n, B = 64 * nb, 64
    g = torch.Generator(device="cuda").manual_seed(nb + d)
    q, k, v = (torch.randn((1, max(heads), n, d), generator=g, device="cuda").to(torch.bfloat16) for _ in range(3))
    rp, ci, _, _ = supports(max(heads), nb, [0, 1, 2, 3, 20, 63, 64], np.random.default_rng(d))
    out = []
    for h in heads:
        r = rp[: h * nb + 1]
        out.append([x[:, : heads[0]] for x in run(gpu_lib, *(x[:, :h].contiguous() for x in (q, k, v)), B, r, ci[: max(r[-1], 1)])])
    for other in out[1:]:
        assert all(torch.equal(a, b) for a, b in zip(out[0], other))
    assert torch.isfinite(out[0][0].float()).all()


# Heads split over the XCDs (7, 17, 33) or taken a few at a time (88), and as they are (8): every block size, the same bits
# for the heads that all grids have
@pytest.mark.parametrize("B,d", [(16, 64), (16, 128), (32, 96), (32, 128), (64, 128), (128, 64)])
def test_work_order_gives_the_same_bits(gpu_lib, B, d):
    nb = 19
    n = 64 * nb if B < 64 else B * nb
    nb = n // B
    g = torch.Generator(device="cuda").manual_seed(B + d)
    q, k, v = (torch.randn((1, 88, n, d), generator=g, device="cuda").to(torch.bfloat16) for _ in range(3))
    rp, ci, _, _ = supports(88, nb, [0, 1, 2, 5, 17], np.random.default_rng(B))
    out = []
    for h in (8, 7, 17, 33, 88):
        r = rp[: h * nb + 1]
        o, lse = run(gpu_lib, *(x[:, :h].contiguous() for x in (q, k, v)), B, r, ci[: r[-1]])
        out.append((o[:, :7], lse[:, :7]))
    for other in out[1:]:
        assert all(torch.equal(a, b) for a, b in zip(out[0], other))


def test_few_heads_at_a_time(gpu_lib):
    """88 heads of 4096 tokens, 32-key blocks: an XCD's keys and values pass 8 MiB, so it takes its 11 heads three at a time;
    a row's output does not depend on it."""
    w, n, B, d = gpu_lib, 4096, 32, 64
    nb = n // B
    g = torch.Generator(device="cuda").manual_seed(5)
    q, k, v = (torch.randn((1, 88, n, d), generator=g, device="cuda").to(torch.bfloat16) for _ in range(3))
    rp, ci, _, _ = supports(88, nb, [1, 2, 9], np.random.default_rng(7))
    whole = run(w, q, k, v, B, rp, ci)
    for h in (0, 30, 87):
        lo, hi = rp[h * nb], rp[(h + 1) * nb]
        one = run(w, *(x[:, h:h + 1].contiguous() for x in (q, k, v)), B, rp[h * nb:(h + 1) * nb + 1] - lo, ci[lo:hi])
        assert torch.equal(one[0][:, 0], whole[0][:, h]) and torch.equal(one[1][:, 0], whole[1][:, h])
