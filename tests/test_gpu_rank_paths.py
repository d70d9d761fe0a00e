"""The replay's and the scorers' paths: vector and scalar loads (array
alignment, odd histories, remainders), the f64 divisions and the integer ones
beyond their range, on both sides of each line.  Bit-exact against the oracle."""
import numpy as np
import pytest

import oracle
from paper_2609_09643_amd import synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def U():
    from paper_2609_09643_amd import unison
    return unison


def shifted(U, a, by):
    """A device copy of `a` that starts `by` elements into its allocation."""
    flat = np.concatenate([np.zeros(by, a.dtype), np.ascontiguousarray(a).reshape(-1)])
    return U._dev(flat)[by:].reshape(a.shape)


GAP_EDGES = np.array([0, 1, 999, 1000, 1001, (1 << 32) - 1, 1 << 32, (1 << 32) * 1000 - 1, (1 << 32) * 1000,
                      (1 << 49) - 1, 1 << 49, (1 << 53) + 1, (1 << 60) + 7, (1 << 63) + 5, (1 << 64) - 1],
                     dtype=np.uint64)


@pytest.mark.parametrize("max_hist,by", [(1, 0), (3, 0), (8, 0), (8, 1), (6, 2)])
@pytest.mark.parametrize("b_g,tau", [(32, 1000), (64, 1), (24, 1_000_000), (48, 1), (49, 7), (50, 3),
                                     (64, 1 << 50), (1, 10)])
def test_ema_replay_paths(U, max_hist, by, b_g, tau):
    rng = np.random.Generator(np.random.PCG64(max_hist * 100 + by + b_g))
    n = 1027
    gaps = (rng.lognormal(np.log(4e9), 2.0, (n, max_hist))).astype(np.uint64)
    wild = rng.random((n, max_hist)) < 0.02           # a few wavefronts meet one
    wild[:512] = False
    gaps[wild] = rng.choice(GAP_EDGES, int(wild.sum()))
    gaps[512 + np.arange(GAP_EDGES.size), 0] = GAP_EDGES
    gaps[:9, 0] = GAP_EDGES[:9]
    n_hist = rng.integers(0, max_hist + 1, n).astype(np.uint8)
    g, gq = U.ema_replay(shifted(U, gaps, by), U._dev(n_hist), b_g, tau)
    og, ogq = oracle.ema_replay(gaps, n_hist, b_g, tau)
    assert np.array_equal(U._host(g, np.uint32), og.view(np.uint32))
    assert np.array_equal(U._host(gq, np.uint64), ogq)


@pytest.mark.parametrize("n", [1, 3, 4, 5, 255, 1023, 1024, 1026])
@pytest.mark.parametrize("by", [0, 1])
def test_scorers_at_sizes_and_alignments(U, n, by):
    rng = np.random.Generator(np.random.PCG64(n))
    turn = rng.integers(0, 256, n).astype(np.uint8)
    done = (rng.random(n) < 0.1).astype(np.uint8)
    g = rng.lognormal(15.0, 2.0, n).astype(np.float32)
    gq = rng.integers(0, 1 << 33, n, dtype=np.uint64)
    d, c = oracle.hazard_counts(synth.hazard_population(3, 128))
    D, N = U._dev(d, np.uint32), U._dev(c, np.uint32)
    x = U.score_fp32(shifted(U, turn, by), shifted(U, g, by), shifted(U, done, by), D, N, 5e8)
    assert np.array_equal(U._host(x, np.uint32), oracle.score_f32(turn, g, done, d, c, 5e8).view(np.uint32))
    for recip in (0, 16):
        y = U.score_fixed(shifted(U, turn, by), shifted(U, gq, by), shifted(U, done, by), D, N, 12,
                          500_000_000, recip)
        assert np.array_equal(U._host(y, np.uint64),
                              oracle.score_fixed(turn, gq, done, d, c, 12, 500_000_000, recip))


@pytest.mark.parametrize("b_h", [6, 11, 12, 13, 16])
@pytest.mark.parametrize("recip", [0, 1, 12, 32])
def test_fixed_score_ranges(U, b_h, recip):
    rng = np.random.Generator(np.random.PCG64(b_h * 40 + recip))
    n = 4096
    gq = rng.integers(0, 1 << 30, n, dtype=np.uint64)
    edges = [v + k for v in (1 << 34, 1 << 38, 1 << 47, 1 << 50, 1 << 53, 1 << 63) for k in (-1, 0, 1)]
    gq[np.arange(len(edges)) * 67 + 500] = np.array(edges, np.uint64)
    gq[4000] = np.uint64((1 << 64) - 1)
    turn = rng.integers(0, 60, n).astype(np.uint8)
    done = (rng.random(n) < 0.02).astype(np.uint8)
    d, c = oracle.hazard_counts(synth.hazard_population(9, 128))
    for p_z in (0, 500_000_000, 1 << 47, (1 << 64) - 1):
        y = U.score_fixed(U._dev(turn), U._dev(gq), U._dev(done), U._dev(d, np.uint32),
                          U._dev(c, np.uint32), b_h, p_z, recip)
        assert np.array_equal(U._host(y, np.uint64), oracle.score_fixed(turn, gq, done, d, c, b_h, p_z, recip)), p_z


@pytest.mark.parametrize("n_per", [2, 5, 63, 64, 66, 127, 128, 130, 191, 192, 193, 254, 255, 256])
@pytest.mark.parametrize("n_snap", [1, 6])
def test_kendall_pairs_at_register_edges(U, n_per, n_snap):
    """Snapshots on one wavefront each: sizes around the register edges, odd
    and even (an even size has a half step), a last block with spare
    wavefronts, ties, infinities, -0 beside +0 and an index out of range; a NaN
    in x is tied with nothing and not greater than anything."""
    rng = np.random.default_rng(31 * n_per + n_snap)
    x = rng.integers(-3, max(2, n_per // 2), (n_snap, n_per)).astype(np.float32)
    y = rng.integers(0, max(2, n_per // 3), (n_snap, n_per)).astype(np.uint64)
    y += np.uint64(2 ** 33) * rng.integers(0, 2, (n_snap, n_per)).astype(np.uint64)
    x[0, ::3] = np.inf
    y[0, ::3] = 2 ** 64 - 1
    x[-1, ::4] = -0.0
    if n_snap > 1:
        x[1] = rng.standard_normal(n_per).astype(np.float32)
    c, t = U.kendall(U._dev(x.ravel()), U._dev(y.ravel()), None, n_snap, n_per)
    oc, ot = oracle.kendall(x, y)
    assert np.array_equal(U._host(c, np.uint64), oc)
    assert np.array_equal(t.cpu().numpy(), ot)
    idx = np.arange(n_snap * n_per, dtype=np.uint32).reshape(n_snap, n_per)[:, ::-1].copy()
    idx[-1, n_per - 1] = n_snap * n_per
    c2, t2 = U.kendall(U._dev(x.ravel()), U._dev(y.ravel()), U._dev(idx))
    assert t2.cpu().numpy()[-1] == 255
    if n_snap > 1:
        oc2, ot2 = oracle.kendall(x[:-1, ::-1].copy(), y[:-1, ::-1].copy())
        assert np.array_equal(U._host(c2, np.uint64)[:-1], oc2)
        assert np.array_equal(t2.cpu().numpy()[:-1], ot2)
    x[0, n_per // 2::5] = np.nan
    c3, _ = U.kendall(U._dev(x.ravel()), U._dev(y.ravel()), None, n_snap, n_per)
    i, j = np.triu_indices(n_per, 1)
    xa, xb, ya, yb = x[0, i], x[0, j], y[0, i], y[0, j]
    tx, ty = xa == xb, ya == yb
    nd = int((~tx & ~ty & ((xa > xb) != (ya > yb))).sum())
    want = [len(i) - nd - int((tx | ty).sum()), nd, int((tx & ~ty).sum()), int((ty & ~tx).sum()), int((tx & ty).sum())]
    assert U._host(c3, np.uint64)[0].tolist() == want


@pytest.mark.parametrize("n_per", [193, 200, 255, 256])
def test_kendall_on_both_sides_of_the_split(U, n_per):
    """Up to 1,024 snapshots of more than 192 entries share a workgroup's
    wavefronts, above that each has one (here with two spare in the last block)."""
    rng = np.random.default_rng(n_per)
    n_snap = 1026
    x = rng.integers(-3, n_per // 2, (n_snap, n_per)).astype(np.float32)
    y = rng.integers(0, n_per // 3, (n_snap, n_per)).astype(np.uint64)
    x[::7, ::3] = np.inf
    x[::5, ::4] = -0.0
    oc, ot = oracle.kendall(x, y)
    for m in (n_snap, 1025, 1024, 3):
        c, t = U.kendall(U._dev(x[:m].ravel()), U._dev(y[:m].ravel()), None, m, n_per)
        assert np.array_equal(U._host(c, np.uint64), oc[:m])
        assert np.array_equal(t.cpu().numpy(), ot[:m])


@pytest.mark.parametrize("more", [-1, 0, 1, 3])
@pytest.mark.parametrize("b_h,recip", [(6, 0), (12, 0), (16, 0), (12, 16), (16, 32)])
def test_fixed_scores_of_pools_with_four_sessions_a_load(U, more, b_h, recip):
    """The integer scorer's vector loads start at 2^21 sessions."""
    n = (1 << 21) + more
    rng = np.random.Generator(np.random.PCG64(b_h + recip))
    gq = rng.integers(0, 1 << 30, n, dtype=np.uint64)
    edges = [v + k for v in (1 << 34, 1 << 38, 1 << 47, 1 << 50, 1 << 53, 1 << 63) for k in (-1, 0, 1)]
    gq[np.arange(len(edges)) * 1067 + 500] = np.array(edges, np.uint64)
    gq[-1] = np.uint64((1 << 64) - 1)
    turn = rng.integers(0, 60, n).astype(np.uint8)
    done = (rng.random(n) < 0.02).astype(np.uint8)
    d, c = oracle.hazard_counts(synth.hazard_population(9, 128))
    y = U.score_fixed(U._dev(turn), U._dev(gq), U._dev(done), U._dev(d, np.uint32), U._dev(c, np.uint32),
                      b_h, 500_000_000, recip)
    assert np.array_equal(U._host(y, np.uint64), oracle.score_fixed(turn, gq, done, d, c, b_h, 500_000_000, recip))


@pytest.mark.parametrize("fixed", [0, 1])
def test_scores_in_place_of_nearly_2_to_the_32_sessions(fixed):
    """The output over the input, with a remainder of the four-session loads whose
    index lies within a grid of 2^32: every session is scored once."""
    import torch
    from paper_2609_09643_amd import unison as U
    n = (1 << 32) - 1001
    head, tail = 1 << 20, 4096
    turn = torch.full((n,), 3, dtype=torch.uint8, device="cuda")
    done = torch.zeros(n, dtype=torch.uint8, device="cuda")
    d, nn = U.hazard_counts(torch.arange(1, 60, dtype=torch.int32, device="cuda"))
    v = torch.empty(n, dtype=torch.int64 if fixed else torch.float32, device="cuda").fill_(5)
    v[:head] = torch.arange(head, device="cuda")
    v[-tail:] = torch.arange(tail, device="cuda")
    ends = torch.cat([v[:head], v[-tail:]]).clone()
    k = ends.numel()
    L = U.lib()
    if fixed:
        want = U.score_fixed(turn[:k].clone(), ends, done[:k].clone(), d, nn, 12, 1000, 0)
        rc = L.unison_score_fixed(U._stream(), n, U._ptr(turn), U._ptr(v), U._ptr(done), U._ptr(d), U._ptr(nn),
                                  12, 1000, 0, U._ptr(v))
    else:
        want = U.score_fp32(turn[:k].clone(), ends, done[:k].clone(), d, nn, 1000.0)
        rc = L.unison_score_fp32(U._stream(), n, U._ptr(turn), U._ptr(v), U._ptr(done), U._ptr(d), U._ptr(nn),
                                 1000.0, U._ptr(v))
    assert rc == 0
    assert torch.equal(v[:head], want[:head])
    assert torch.equal(v[-tail:], want[head:])
    assert bool((v[head:-tail:4097] == v[head]).all())
    del v, turn, done
    torch.cuda.empty_cache()
