"""Pins of the oracle's lattice decoders and constants (CPU only).

The decoders are checked against enumeration of lattice points written here
from the membership constraints of Sec. 4.6 (not from the decoders), the
lattice facts the paper and the literature fix (minimum norms, kissing
numbers, covolumes, theta-series shells), and Monte-Carlo normalized second
moments against Tab. lattice-constants.
"""
import itertools

import numpy as np
import pytest

from oracle import oracle as O

LATS = [O.E8, O.D4, O.A2, O.Z]
# covering radius of each integer realization (2E8: 2, D4: 1, A2: 2/sqrt3, Z: 1/2)
RHO = {O.E8: 2.0, O.D4: 1.0, O.A2: 2.0 / np.sqrt(3.0), O.Z: 0.5}


def member(lat, c):
    """Membership in the integer realization, from Sec. 4.6's constraints."""
    c = np.asarray(c, dtype=np.int64)
    if lat == O.E8:
        cb = c[..., :1] & 1
        same = np.all(((c - cb) & 1) == 0, axis=-1)
        s = (c - cb) // 2
        return same & ((s.sum(axis=-1) & 1) == 0)
    if lat == O.D4:
        return (c.sum(axis=-1) & 1) == 0
    if lat == O.A2:
        return ((c[..., 0] + c[..., 1]) & 1) == 0
    return np.ones(c.shape[:-1], dtype=bool)


def points(lat, c):
    return O.lattice_points(lat, c)


def enumerate_box(lat, lo, hi):
    """All integer codes in the box [lo, hi] (per coordinate) that are members."""
    m = O.DIM[lat]
    g = np.arange(lo[0], hi[0] + 1, dtype=np.int64)[:, None]
    for i in range(1, m):
        ax = np.arange(lo[i], hi[i] + 1, dtype=np.int64)
        g = np.concatenate([np.repeat(g, ax.size, axis=0), np.tile(ax, g.shape[0])[:, None]], axis=1)
    return g[member(lat, g)]


def shell(lat, max_norm2):
    """Lattice vectors (as codes) of squared Euclidean norm <= max_norm2,
    enumerated over Z^m coordinate by coordinate with the partial norm pruned."""
    m = O.DIM[lat]
    w = np.array([3.0 if (lat == O.A2 and i == 0) else 1.0 for i in range(m)])  # |point_i|^2 = w_i c_i^2
    r = int(np.floor(np.sqrt(max_norm2)))
    g = np.zeros((1, 0), dtype=np.int64)
    part = np.zeros(1)
    for i in range(m):
        ax = np.arange(-r, r + 1, dtype=np.int64)
        g = np.concatenate([np.repeat(g, ax.size, axis=0), np.tile(ax, g.shape[0])[:, None]], axis=1)
        part = np.repeat(part, ax.size) + w[i] * np.tile(ax, part.size) ** 2
        keep = part <= max_norm2 + 1e-9
        g, part = g[keep], part[keep]
    return g[member(lat, g)]


def test_lattice_facts():
    # P4: E8 min norm 2 and kissing number 240 (bare scaling; 8 and 240 in
    # 2E8), D4 min norm 2 with 24 minimal vectors, A2 min distance 2 with 6,
    # Z: 2.  The next shells of E8 (2160) and D4 (24) as well.
    def counts(lat, lim):
        v = shell(lat, lim)
        n2 = np.round((points(lat, v) ** 2).sum(axis=1), 9)
        vals, cnt = np.unique(n2, return_counts=True)
        return dict(zip(vals.tolist(), cnt.tolist()))

    assert counts(O.E8, 16) == {0.0: 1, 8.0: 240, 16.0: 2160}
    assert counts(O.D4, 4) == {0.0: 1, 2.0: 24, 4.0: 24}
    assert counts(O.A2, 4) == {0.0: 1, 4.0: 6}
    assert counts(O.Z, 1) == {0.0: 1, 1.0: 2}


BASES = {
    # E8 basis (Conway & Sloane): 2e1, e2-e1, ..., e7-e6, (1/2)^8; doubled -> 2E8.
    O.E8: 2.0 * np.array([[2, 0, 0, 0, 0, 0, 0, 0],
                          [-1, 1, 0, 0, 0, 0, 0, 0],
                          [0, -1, 1, 0, 0, 0, 0, 0],
                          [0, 0, -1, 1, 0, 0, 0, 0],
                          [0, 0, 0, -1, 1, 0, 0, 0],
                          [0, 0, 0, 0, -1, 1, 0, 0],
                          [0, 0, 0, 0, 0, -1, 1, 0],
                          [0.5] * 8], dtype=np.float64),
    O.D4: np.array([[1, -1, 0, 0], [0, 1, -1, 0], [0, 0, 1, -1], [0, 0, 1, 1]], dtype=np.float64),
    O.A2: np.array([[np.sqrt(3.0), 1.0], [0.0, 2.0]]),
    O.Z: np.array([[1.0]]),
}


@pytest.mark.parametrize("lat", LATS)
def test_basis_and_covolume(lat):
    B = BASES[lat]
    assert abs(abs(np.linalg.det(B)) - O.covolume(lat)) < 1e-9 * O.covolume(lat)
    codes = B.copy()
    if lat == O.A2:
        codes[:, 0] /= np.sqrt(3.0)
    codes = np.round(codes).astype(np.int64)
    assert np.all(member(lat, codes))


@pytest.mark.parametrize("lat", LATS)
def test_decoder_matches_plain_enumeration(lat):
    # P3, tiny inputs: every lattice point within the covering radius of z is
    # enumerated from the membership constraints; the decoder's point must be
    # at the minimum distance.
    rng = np.random.default_rng(100 + lat)
    m = O.DIM[lat]
    nz = 16 if lat == O.E8 else 48
    z = (rng.standard_normal((nz, m)) * 3.0).astype(np.float32)
    c = O.quantize(lat, z)
    assert np.all(member(lat, c))
    for i in range(nz):
        zi = z[i].astype(np.float64)
        if lat == O.A2:
            lo = [int(np.floor(zi[0] / np.sqrt(3) - 2)), int(np.floor(zi[1] - 2))]
            hi = [int(np.ceil(zi[0] / np.sqrt(3) + 2)), int(np.ceil(zi[1] + 2))]
        else:
            lo = [int(np.floor(v - RHO[lat])) for v in zi]
            hi = [int(np.ceil(v + RHO[lat])) for v in zi]
        cand = enumerate_box(lat, lo, hi)
        d = ((points(lat, cand) - zi) ** 2).sum(axis=1)
        dc = ((points(lat, c[i:i + 1]) - zi) ** 2).sum()
        assert dc <= d.min() + 1e-5, (i, zi, c[i], cand[d.argmin()])


@pytest.mark.parametrize("lat", LATS)
def test_decoder_exact_nearest_by_shells(lat):
    # P3, bulk: for 1e5 z, |z - Q(z)| <= rho and no Q(z) + v is closer for any
    # lattice vector v with |v| <= 2 rho (which covers every competitor once
    # the first condition holds).  Near-ties within fp32 rounding are allowed.
    rng = np.random.default_rng(200 + lat)
    m = O.DIM[lat]
    n = 100000
    z = (rng.standard_normal((n, m)) * 4.0).astype(np.float32)
    c = O.quantize(lat, z)
    assert np.all(member(lat, c))
    p = points(lat, c)
    zd = z.astype(np.float64)
    d0 = ((zd - p) ** 2).sum(axis=1)
    assert np.sqrt(d0.max()) <= RHO[lat] + 1e-5
    V = points(lat, shell(lat, (2 * RHO[lat]) ** 2 + 1e-9))
    vv = (V ** 2).sum(axis=1)
    e = zd - p
    worst = 0.0
    for a in range(0, n, 20000):
        # |e - v|^2 = |e|^2 - (2 <e, v> - |v|^2): the best competitor's gain
        gain = (2.0 * (e[a:a + 20000] @ V.T) - vv[None, :]).max(axis=1)
        worst = max(worst, gain.max())
    assert worst <= 1e-4


@pytest.mark.parametrize("lat", LATS)
def test_idempotent_and_equivariant(lat):
    rng = np.random.default_rng(300 + lat)
    m = O.DIM[lat]
    lam = O.unstrip(lat, rng.integers(0, 40, size=(2000, m)).astype(np.uint32))
    assert np.all(member(lat, lam))
    lam_pts = points(lat, lam).astype(np.float32)
    assert np.array_equal(O.quantize(lat, lam_pts), lam)
    # Q(z + lambda) = Q(z) + lambda away from cell boundaries (integer shifts only,
    # so z + lambda stays exact in fp32 for E8, D4, Z; A2 shifts along nx only).
    z = (rng.standard_normal((2000, m)) * 3.0).astype(np.float32)
    shift = lam.copy()
    if lat == O.A2:
        shift[:, 0] = 0
        shift[:, 1] = 2 * (shift[:, 1] // 2)
    cz = O.quantize(lat, z)
    mg = O.margins(lat, z, cz)
    zs = (z + points(lat, shift).astype(np.float32)).astype(np.float32)
    czs = O.quantize(lat, zs)
    ok = mg > 1e-3
    assert ok.mean() > 0.9
    assert np.array_equal(czs[ok], (cz + shift)[ok])


def test_margin_sign():
    # The margin is positive inside the chosen cell and negative if the code
    # is moved to a neighbour.
    rng = np.random.default_rng(5)
    for lat in LATS:
        m = O.DIM[lat]
        z = (rng.standard_normal((500, m)) * 2).astype(np.float32)
        c = O.quantize(lat, z)
        assert np.all(O.margins(lat, z, c) > -1e-6)
        v = shell(lat, {O.E8: 8, O.D4: 2, O.A2: 4, O.Z: 1}[lat])
        v = v[np.any(v != 0, axis=1)][0]
        assert np.all(O.margins(lat, z, c + v) < 0)


PAPER_G = {O.Z: 0.0833, O.A2: 0.0802, O.D4: 0.0766, O.E8: 0.0717}


@pytest.mark.parametrize("lat", LATS)
def test_normalized_second_moment_monte_carlo(lat):
    # P5 / App. A sampler: T ~ U[0,1)^m, Y = sum T_i b_i (a point of the
    # fundamental parallelepiped), U = Y - Q(Y) is uniform on the Voronoi
    # cell; G = E|U|^2 / (m V^(2/m)) must match Tab. lattice-constants.
    rng = np.random.default_rng(400 + lat)
    m = O.DIM[lat]
    n = 400000
    Y = rng.random((n, m)) @ BASES[lat]
    Yf = Y.astype(np.float32)
    c = O.quantize(lat, Yf)
    U = Yf.astype(np.float64) - points(lat, c)
    G = (U ** 2).sum(axis=1).mean() / (m * O.covolume(lat) ** (2.0 / m))
    assert abs(G - PAPER_G[lat]) / PAPER_G[lat] < 0.005
    assert abs(G - O.nsm(lat)) / O.nsm(lat) < 0.005
    # the printed table values are the exact ones rounded to 4 digits
    assert round(O.nsm(lat), 4) == PAPER_G[lat]
    if lat == O.E8:
        # App. A: sigma^2_Vor(E8) ~ 0.287 in this scaling
        assert abs((U ** 2).mean() - 0.287) < 0.002


def test_gaps_and_gains_match_paper():
    # Tab. lattice-constants: gap to Shannon 10 log10(2 pi e G); Sec. 3.2
    # granular gains over Z of 0.17 / 0.37 / 0.65 dB.
    gap = {lat: 10 * np.log10(2 * np.pi * np.e * O.nsm(lat)) for lat in LATS}
    # (the table prints A2 as 1.36 where the exact G gives 1.366)
    for l, v in zip((O.Z, O.A2, O.D4, O.E8), (1.53, 1.36, 1.17, 0.88)):
        assert abs(gap[l] - v) < 0.011
    gain = {lat: 10 * np.log10(O.nsm(O.Z) / O.nsm(lat)) for lat in LATS}
    assert [round(gain[l], 2) for l in (O.A2, O.D4, O.E8)] == [0.17, 0.37, 0.65]


@pytest.mark.parametrize("step", [2.0 ** -22, 2.0 ** -6, 2.0 ** -2, 2.0 ** -1, 1.0])
def test_e8_box_point_from_even_errors(step):
    """The E8 dither point's closed form on its box against the general decoder: the odd coset's
    errors are ea - sign(ea), D's sign decides away from ties, one moved coordinate ends it.  The
    coarse steps make ties and equal magnitudes; blocks in the tie band (or with every |ea| = 1) are
    the two-coset form's and are left out, as the kernels do."""
    rng = np.random.default_rng(int(1 / step))
    n = int(4 / step)
    b = (rng.integers(0, n, (200000, 8)) * step - 2.0).astype(np.float32)
    u = b - O.quantize(O.E8, b).astype(np.float32)
    t = b * np.float32(0.5) + np.float32(12582912.0)
    ea = b - np.float32(2.0) * (t - np.float32(12582912.0))
    assert not np.any(np.signbit(ea) & (ea == 0))
    a = np.abs(ea)
    odd_a = np.bitwise_xor.reduce(t.view(np.uint32), axis=1) & 1 == 1
    odd_b = np.signbit(b).sum(axis=1) % 2 == 1
    mx, mn = a.max(axis=1), a.min(axis=1)
    D = 8 - 2 * a.astype(np.float64).sum(axis=1) + np.where(odd_b, 4 * mn, 0) - np.where(odd_a, 4 - 4 * mx, 0)
    ok = (np.abs(D) >= 2.0 ** -13) & (mn < 1)
    even = D > 0
    target = np.where(even, np.where(odd_a, mx, 2), np.where(odd_b, mn, 2))
    add = np.repeat(np.where(even, 0.0, -1.0)[:, None], 8, axis=1)
    hit = a == target[:, None]
    rows = np.nonzero(hit.any(axis=1))[0]
    add[rows, hit[rows].argmax(axis=1)] = np.where(even[rows], -2.0, 1.0)
    v = ea + (add * np.where(np.signbit(ea), -1, 1)).astype(np.float32)
    assert ok.sum() > (1000 if step < 1 else 0)
    assert np.array_equal(u[ok], v[ok])
