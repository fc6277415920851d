"""The in-place stage plan of the passes at the lengths without instantiated
kernels (csrc/fft_any.h), restated on the CPU (no GPU): at every length
2^a 3^b 5^c 7^d up to 1024 the plan's radices multiply to the length, a
workgroup fits its limits, the multiply-high divisions are exact over the
indices they meet, every stage's butterflies touch each slot once, twiddle
indices stay in the table, and the stages with the kernels' indexing give
numpy's FFT: decimation in frequency to the slots of block_freq, decimation
in time from the slots of slot_of, and an axis-3 pass (pairwise packing, the
last inverse stage, the mask and the first forward stage on the same values,
pairwise unpacking) numpy's irfft / mask / rfft; so does that of an odd N3,
which takes the rows two by two, with the mask read from its words, over
several workgroups and a last row without a partner."""
import numpy as np
import pytest

RADICES = (10, 9, 8, 7, 6, 5, 4, 3, 2)
MAX_THREADS = 512


def smooth(n):
    for f in (2, 3, 5, 7):
        while n % f == 0:
            n //= f
    return n == 1


LENGTHS = [n for n in range(1, 1025) if smooth(n)]


def plan(L):
    best = None

    def search(rest, top, cur):
        nonlocal best
        if rest == 1:
            if cur and (best is None or (len(cur), sum(cur)) < (len(best), sum(best))):
                best = list(cur)
            return
        if len(cur) == 5 or (best and len(cur) >= len(best)):
            return
        for r in RADICES:
            if r <= top and rest % r == 0:
                search(rest // r, r, cur + [r])

    search(L, 10, [])
    st = best or [1]
    return st if len(st) > 1 else [1] + st


def shape(L, st, w, pencils=None, lowest=2):
    """Pencils per workgroup and threads per pencil; fewer pencils (not below
    2^lowest) where fewer than 128 workgroups would take them all."""
    least = -(-L // max(st))
    lg = 4 if w == 8 else 3
    while (1 << lg) * least < 64 and lg < 6:
        lg += 1
    while pencils is not None and lg > lowest and -(-pencils >> lg) < 128 and (1 << lg) // 2 * least >= 64:
        lg -= 1
    tm = 1 << lg
    unit = 64 // tm
    return tm, min(-(-least // unit) * unit, MAX_THREADS // tm)


def magic(d):
    return -(-(1 << 32) // d)


def div(n, d):
    assert np.all(n < 65536) and 2 <= d <= 1024
    q = (n.astype(np.uint64) * np.uint64(magic(d))) >> np.uint64(32)
    assert np.array_equal(q, n // d)
    return q.astype(np.int64)


def block_freq(b, st):
    f = np.zeros_like(b)
    for s in range(len(st) - 2, 0, -1):
        q = div(b, st[s])
        f = (b - q * st[s]) + st[s] * f
        b = q
    return b + st[0] * f


def slot_of(n, st):
    o = np.zeros_like(n)
    for r in st[:-1]:
        q = n if r == 1 else div(n, r)
        o = o * r + (n - q * r)
        n = q
    return o * st[-1] + n


def stage(a, L, st, s, sgn, time):
    """Stage s in place (decimation in time when `time`)."""
    B = L // int(np.prod(st[:s], dtype=np.int64))
    R = st[s]
    ms, step = B // R, L // B
    b = np.arange(L // R)
    blk = np.zeros_like(b) if s == 0 else (b if ms == 1 else div(b, ms))
    j = b - blk * ms
    q = np.arange(R)
    at = (blk * ms * R + j)[:, None] + q[None, :] * ms
    assert np.array_equal(np.sort(at.ravel()), np.arange(L))
    ti = j[:, None] * step * q[None, :]
    assert ti.min() >= 0 and ti.max() < max(L, 1)
    tw = np.exp(sgn * 2j * np.pi * ti / L)
    dft = np.exp(sgn * 2j * np.pi * np.outer(q, q) / R)
    v = a[at]
    v = (v * tw) @ dft if time else (v @ dft) * tw
    a[at] = v


@pytest.mark.parametrize("L", LENGTHS)
def test_plan_and_transforms(L):
    st = plan(L)
    assert int(np.prod(st)) == L and 2 <= len(st) <= 5 and max(st) <= 10
    for w in (8, 16):
        tm, nt = shape(L, st, w)
        assert tm * nt <= MAX_THREADS and (tm * nt) % 64 == 0 and tm >= 4
        assert (tm + 1) * L * w <= 163840                       # the strided tile and its twiddles
        if L <= 512 or L % 2:   # an axis-3 pass (N3 = 2 L, or an odd N3 = L): tile, twiddles and mask words
            assert L * (tm + 2) * w + 4 * (2 * tm * L // 32 + 2) <= 163840
            assert 2 * tm * L < 65536                           # the indices of its runs
        for pencils in (1, 7, 60, 127 * tm, 127 * tm + 1, 1000, 10 ** 6):
            for lowest in (0, 2):   # row pairs, strided passes
                fm, ft = shape(L, st, w, pencils, lowest)
                assert (1 << lowest) <= fm <= tm and (fm == tm or -(-pencils // (2 * fm)) < 128)
                assert fm * ft <= MAX_THREADS and (fm * ft) % 64 == 0 and ft >= min(nt, -(-L // max(st)))
    rng = np.random.default_rng(L)
    x = rng.standard_normal(L) + 1j * rng.standard_normal(L)
    n = np.arange(L)
    slots = slot_of(n, st)
    assert np.array_equal(np.sort(slots), n)
    nbf = L // st[-1]
    freq = (block_freq(np.arange(nbf), st)[:, None] + nbf * np.arange(st[-1])[None, :]).ravel()
    assert np.array_equal(freq[slots], n)
    for sgn in (-1, 1):
        ref = np.fft.fft(x) if sgn < 0 else np.fft.ifft(x) * L
        a = x.copy()
        for s in range(len(st)):
            stage(a, L, st, s, sgn, False)
        assert np.linalg.norm(a[slots] - ref) <= 1e-12 * np.linalg.norm(ref)
        a = np.empty_like(x)
        a[slots] = x
        for s in range(len(st) - 1, -1, -1):
            stage(a, L, st, s, sgn, True)
        assert np.linalg.norm(a - ref) <= 1e-12 * np.linalg.norm(ref)


@pytest.mark.parametrize("L", [n for n in LENGTHS if 2 <= n <= 512])
def test_axis3_pass(L):
    st = plan(L)
    N = 2 * L
    rng = np.random.default_rng(N)
    X = rng.standard_normal(L) + 1j * rng.standard_normal(L)   # slot 0: DC and Nyquist
    mask = rng.random(N) < 0.7
    w = np.exp(-2j * np.pi * np.arange(L) / N)
    a = np.empty(L, np.complex128)
    r2 = np.sqrt(2.0)
    a[0] = r2 * (X[0].real + X[0].imag) + 1j * r2 * (X[0].real - X[0].imag)
    e = np.arange(1, L // 2 + 1)
    sm, d = X[e] + X[L - e].conj(), X[e] - X[L - e].conj()
    it = 1j * w[e].conj() * d
    a[e] = sm + it
    a[L - e] = (sm - it).conj()
    for s in range(len(st) - 1):
        stage(a, L, st, s, +1, False)
    R = st[-1]
    nbf = L // R
    q = np.arange(R)
    at = np.arange(nbf)[:, None] * R + q[None, :]
    nat = block_freq(np.arange(nbf), st)[:, None] + nbf * q[None, :]
    z = a[at] @ np.exp(2j * np.pi * np.outer(q, q) / R)
    z = z.real * mask[2 * nat] + 1j * z.imag * mask[2 * nat + 1]
    a[at] = z @ np.exp(-2j * np.pi * np.outer(q, q) / R)
    for s in range(len(st) - 2, -1, -1):
        stage(a, L, st, s, -1, True)
    rn = 1.0 / np.sqrt(N)
    Y = np.empty(L, np.complex128)
    Y[0] = ((a[0].real + a[0].imag) + 1j * (a[0].real - a[0].imag)) * (rn * rn / r2)
    e = np.arange(1, L // 2 + 1)
    sm, d = a[e] + a[L - e].conj(), a[e] - a[L - e].conj()
    it = -1j * w[e] * d
    Y[e], Y[L - e] = (sm + it) * (rn * rn / 2), (sm - it).conj() * (rn * rn / 2)
    half = np.empty(L + 1, np.complex128)
    half[0], half[L], half[1:L] = X[0].real, X[0].imag, X[1:] / r2
    ref = np.fft.rfft(np.where(mask, np.fft.irfft(half, N, norm="ortho"), 0.0), norm="ortho")
    got = np.empty(L + 1, np.complex128)
    got[0], got[L], got[1:L] = Y[0].real, Y[0].imag, Y[1:] / r2
    assert np.linalg.norm(got - ref) <= 1e-12 * np.linalg.norm(ref)


@pytest.mark.parametrize("L", [n for n in LENGTHS if n >= 3 and n % 2])
def test_odd_axis3_pass(L):
    """k_axis3_odd: three passes (inverse alone, both with the mask, forward
    alone) over seven rows in workgroups of two pairs."""
    st, M, rows, TM = plan(L), (L + 1) // 2, 7, 2
    rng = np.random.default_rng(L)
    X = rng.standard_normal((rows, M)) + 1j * rng.standard_normal((rows, M))   # sqrt2 times the half spectra,
    X[:, 0] = X[:, 0].real                                                     # the real value of e = 0 once
    mask = rng.random(rows * L) < 0.7
    words = np.zeros(rows * L // 32 + 1, np.uint32)
    np.bitwise_or.at(words, np.nonzero(mask)[0] >> 5, np.uint32(1) << (np.nonzero(mask)[0] & 31).astype(np.uint32))
    real = rng.standard_normal((rows, L))
    R = st[-1]
    nbf, q = L // R, np.arange(R)
    at = np.arange(nbf)[:, None] * R + q[None, :]
    nat = block_freq(np.arange(nbf), st)[:, None] + nbf * q[None, :]
    slots = slot_of(np.arange(L), st)
    r2, rn = np.sqrt(2.0), 1.0 / np.sqrt(L)
    back = np.full((rows, L), np.nan)
    full, fwd = (np.full((rows, M), np.nan, np.complex128) for _ in range(2))
    zero = np.zeros(M, np.complex128)
    for group in range(-(-rows // (2 * TM))):
        row0 = 2 * TM * group
        nrow = min(2 * TM, rows - row0)
        bit0 = row0 * L
        nw = ((bit0 + nrow * L - 1) >> 5) - (bit0 >> 5) + 1
        assert nw <= 2 * TM * L // 32 + 2 and (bit0 >> 5) + nw <= words.size
        mw = words[bit0 >> 5:(bit0 >> 5) + nw]
        for p in range(TM):
            on = [2 * p < nrow, 2 * p + 1 < nrow]
            x, y = (X[row0 + 2 * p + k] if on[k] else zero for k in (0, 1))
            for masked in (False, True):
                a = np.empty(L, np.complex128)
                a[0] = r2 * x[0].real + 1j * r2 * y[0].real
                e = np.arange(1, M)
                a[e] = (x[e].real - y[e].imag) + 1j * (x[e].imag + y[e].real)
                a[L - e] = (x[e].real + y[e].imag) + 1j * (y[e].real - x[e].imag)
                for s in range(len(st) - 1):
                    stage(a, L, st, s, +1, False)
                v = a[at] @ np.exp(2j * np.pi * np.outer(q, q) / R)
                if not masked:
                    a[at] = v
                    z = a[slots] * (rn / r2)
                    if on[0]:
                        back[row0 + 2 * p] = z.real
                    if on[1]:
                        back[row0 + 2 * p + 1] = z.imag
                    continue
                ba = (bit0 & 31) + 2 * p * L + nat
                keep = [((mw[(ba + k * L) >> 5] >> ((ba + k * L) & 31).astype(np.uint32)) & 1) if on[k] else 0 for k in (0, 1)]
                a[at] = (v.real * keep[0] + 1j * v.imag * keep[1]) @ np.exp(-2j * np.pi * np.outer(q, q) / R)
                for s in range(len(st) - 2, -1, -1):
                    stage(a, L, st, s, -1, True)
                unpack(a, L, M, on, row0 + 2 * p, full, rn * rn / r2, rn * rn / 2)
            a = np.empty(L, np.complex128)
            a[slots] = (real[row0 + 2 * p] if on[0] else 0.0) + 1j * (real[row0 + 2 * p + 1] if on[1] else 0.0)
            for s in range(len(st) - 1, -1, -1):
                stage(a, L, st, s, -1, True)
            unpack(a, L, M, on, row0 + 2 * p, fwd, rn, rn / r2)
    half = X / r2
    half[:, 0] = X[:, 0]
    sig = np.fft.irfft(half, L, norm="ortho")
    spec = np.fft.rfft(np.where(mask.reshape(rows, L), sig, 0.0), norm="ortho")
    spec[:, 1:] *= r2
    spec2 = np.fft.rfft(real, norm="ortho")
    spec2[:, 1:] *= r2
    for got, ref in ((back, sig), (full, spec), (fwd, spec2)):
        assert np.linalg.norm(got - ref) <= 1e-12 * np.linalg.norm(ref)


def unpack(a, L, M, on, row, out, dc, ac):
    e = np.arange(1, M)
    y, z = a[e], a[L - e]
    if on[0]:
        out[row, 0] = a[0].real * dc
        out[row, e] = ((y.real + z.real) + 1j * (y.imag - z.imag)) * ac
    if on[1]:
        out[row + 1, 0] = a[0].imag * dc
        out[row + 1, e] = ((y.imag + z.imag) + 1j * (z.real - y.real)) * ac
