"""Selection where its paths meet: sums by digit against ranked rows (masses
whose fp64 sums round, negative and infinite ones, ties at the cut, light
masses few and many and at the threshold's last bit), chunk edges of the CSR kernel, and row counts past the
limit of its sums.  Bit for bit the oracle's."""

import numpy as np
import pytest
import torch

from oracle import wise_oracle as O

pytestmark = pytest.mark.gpu


def masses(kind, rows, nb, rng):
    x = rng.random((rows, nb)).astype(np.float32)
    if kind == "wide":          # exponents over 2^-60 .. 1: light masses in most rows
        x *= np.exp2(-rng.integers(0, 60, (rows, nb))).astype(np.float32)
    elif kind == "light":       # one heavy block, the others below 2^-32: more than 64 light ones where nb allows
        x *= np.float32(2.0 ** -33)
        x[np.arange(rows), rng.integers(0, nb, rows) * (np.arange(rows) % nb) // nb] = 1.0
    elif kind == "ties":        # few distinct values, zeros among them
        x = rng.integers(0, 4, (rows, nb)).astype(np.float32) * np.float32(0.125)
    elif kind == "denormal":
        x = (rng.integers(0, 3, (rows, nb)) * np.float32(1e-45)).astype(np.float32)
    elif kind == "odd":         # negative and infinite masses, minus zero
        x[::3, ::2] *= -1
        x[1::5, 1::3] = -0.0
        x[2::7, 0] = np.inf
    elif kind == "peaked":
        x = (x ** 40).astype(np.float32)
    elif kind == "edge":        # tau 0.5: the threshold is the first mass, or one rounding above it, by the sum of 128 light ones
        x[:] = 0
        x[:, 0] = 0.5 + 2.0 ** -23
        x[:, 1:2] = 0.5 - 2.0 ** -23
        x[:, 2:130] = 2.0 ** -29
        x[1::2, 60:61] *= np.float32(1 + 2.0 ** -23)
        x[2::3, 90:91] *= np.float32(1 + 2.0 ** -21)
    elif kind == "mixed":       # a few heavy ones, light ones of every size below
        x = np.where(rng.random((rows, nb)) < 0.03, x, x * np.exp2(-rng.integers(27, 70, (rows, nb)))).astype(np.float32)
    return x


@pytest.mark.parametrize("kind", ["plain", "wide", "light", "ties", "denormal", "odd", "peaked", "edge", "mixed"])
@pytest.mark.parametrize("nb", [1, 2, 64, 127, 129, 300, 1024])
def test_selection_paths(gpu_lib, kind, nb):
    w = gpu_lib
    heads = 3 if nb < 1024 else 1
    rng = np.random.default_rng(nb * 31 + len(kind))
    acc = masses(kind, heads * nb, nb, rng).reshape(1, heads, nb, nb)
    s = w.make_shape(1, heads, 64 * nb, 64, 64)
    sched = w.Schedule(s)
    for tau, flags in ((0.95, 3), (0.5, 0), (1.0, 0), (0.9999999, 2)):
        tau = float(np.float32(tau))
        sched.select(torch.from_numpy(acc).cuda(), tau, flags)
        torch.cuda.synchronize()
        with np.errstate(invalid="ignore"):
            rp, ci = O.select_support(acc.astype(np.float64), tau, flags)
        assert np.array_equal(sched.row_ptr.cpu().numpy(), rp), (kind, nb, tau, flags)
        assert np.array_equal(sched.col_idx[: len(ci)].cpu().numpy(), ci), (kind, nb, tau, flags)
        assert np.array_equal(sched.row_order.cpu().numpy(), O.schedule_order(rp, nb))


# one head, several whole heads and part of a head per group of the CSR kernel; a last group that is not full
@pytest.mark.parametrize("heads,nb", [(8200, 16), (70, 3), (1, 1024), (512, 1), (1300, 1), (1025, 2), (5000, 3), (1600, 42), (1600, 43), (600, 63),
                                      (1030, 64), (520, 65), (2, 127), (2, 128), (2, 129), (70000, 2), (1 << 22, 1), (8200, 129)])
def test_csr_of_many_rows(gpu_lib, heads, nb):
    """Row counts 4 does not divide, 4194304 heads (a 1024-thread group for each would be more than a
    grid holds) and 1057800 rows of two groups a head (both past the limit of the sums in the CSR kernel)."""
    w = gpu_lib
    rng = np.random.default_rng(heads)
    s = w.make_shape(1, heads, 64 * nb, 64, 64)
    words = w.wise_mask_words(s)
    m = rng.integers(0, 1 << 63, (heads * nb, words), dtype=np.int64)
    sched = w.Schedule(s)
    sched.from_masks(torch.from_numpy(m).cuda(), 1, 3)
    torch.cuda.synchronize()
    bits = np.unpackbits(m.view(np.uint8).reshape(heads * nb, words * 8), axis=1, bitorder="little")[:, :nb].astype(bool)
    qb = np.arange(heads * nb) % nb
    bits &= np.arange(nb)[None, :] <= qb[:, None]
    bits[:, 0] = True
    bits[np.arange(heads * nb), qb] = True
    rp = np.concatenate(([0], bits.sum(1).cumsum())).astype(np.int32)
    assert np.array_equal(sched.row_ptr.cpu().numpy(), rp)
    assert np.array_equal(sched.col_idx[: rp[-1]].cpu().numpy(), np.nonzero(bits)[1])
    assert np.array_equal(sched.row_order.cpu().numpy(), O.schedule_order(rp, nb))


@pytest.mark.parametrize("kind", ["plain", "wide", "ties", "denormal", "odd", "peaked"])
@pytest.mark.parametrize("nb", [11, 12, 13, 14])
def test_step_around_the_ranked_rows(gpu_lib, kind, nb):
    """Rows of up to 12 candidates are ranked, longer ones cut by digits."""
    w = gpu_lib
    heads = 40
    acc = masses(kind, heads * nb, nb, np.random.default_rng(nb)).reshape(1, heads, nb, nb)
    s = w.make_shape(1, heads, 64 * nb, 64, 64)
    mask = torch.zeros(heads * nb, 1, dtype=torch.int64, device="cuda")
    for tau in (0.3, 0.95, 1.0):
        tau = float(np.float32(tau))
        w.wise_select_step(s, torch.from_numpy(acc).cuda(), tau, mask)
        torch.cuda.synchronize()
        with np.errstate(invalid="ignore"):
            rp, ci = O.select_support(acc.astype(np.float64), tau, 0)
        got = np.unpackbits(mask.cpu().numpy().view(np.uint8), axis=1, bitorder="little")[:, :nb]
        want = np.zeros_like(got)
        want[np.repeat(np.arange(heads * nb), np.diff(rp)), ci] = 1
        assert np.array_equal(got, want), (kind, nb, tau)
