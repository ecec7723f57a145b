"""16- and 32-key-block rows whose ids come 64 at a time: row lengths around that
batch, one and two blocks in the last tile, ids to skip at batch edges, and
rows with none, against the oracle."""

import numpy as np
import pytest
import torch

from oracle import wise_oracle as O
from parity_util import assert_attn, assert_lse, f64

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B", [16, 32])
@pytest.mark.parametrize("d,kv_heads", [(64, 1), (96, 2), (128, 2)])
def test_one_wave_rows_id_batches(gpu_lib, d, kv_heads, B):
    w = gpu_lib
    n, h = 132 * B, 2
    nb = n // B
    g = torch.Generator().manual_seed(d)
    q = (torch.randn((1, h, n, d), generator=g) * 1.5).to(torch.bfloat16)
    k, v = (torch.randn((1, kv_heads, n, d), generator=g).to(torch.bfloat16) for _ in range(2))
    rng = np.random.default_rng(d)
    rp, ci, clean_rp, clean_ci = [0], [], [0], []
    for r in range(h * nb):
        qb = r % nb
        size = min(qb + 1, int(rng.choice([0, 1, 2, 63, 64, 65, 127, 128, 129, 132])))
        row = sorted(rng.choice(qb + 1, size=size, replace=False).tolist())
        past = [i for i in range(qb + 1, min(qb + 1 + int(rng.integers(0, 70)), nb))]   # skipped
        ci.extend(row + past)
        rp.append(len(ci))
        clean_ci.extend(row)
        clean_rp.append(len(clean_ci))
    s = w.make_shape(1, h, n, d, B, kv_heads=kv_heads)
    o = torch.empty_like(q, device="cuda")
    lse = torch.empty((1, h, n), device="cuda")
    to = lambda x: torch.from_numpy(np.asarray(x, np.int32)).cuda()  # noqa: E731
    w.wise_sparse_attn(s, q.cuda(), k.cuda(), v.cuda(), to(rp), to(ci), None, o, lse)
    torch.cuda.synchronize()
    o_ref, l_ref = O.sparse_attention(f64(q), O.expand_kv(f64(k), h), O.expand_kv(f64(v), h),
                                      np.asarray(clean_rp, np.int32), np.asarray(clean_ci, np.int32), B)
    assert_attn(o, o_ref, f"d={d}")
    assert_lse(lse, l_ref)
