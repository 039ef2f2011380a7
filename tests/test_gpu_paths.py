"""Kernel paths chosen by size, precision and fifth-dimension extent, against the oracle at the edges
of their ranges.  Tolerances are those of one application in the storage precision (FP64 1e-12,
FP32 1e-5, FP16 4e-3, BF16 3e-2 of the largest component), as for every operator test here."""
import numpy as np
import pytest

import synth
from gpu_helpers import PREC_TOL, gpu_ctx, mask, rel_err

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def env():
    return gpu_ctx()


@pytest.mark.parametrize("Ls", [8, 16, 32])
@pytest.mark.parametrize("prec", ["fp64", "fp32", "fp16", "bf16"])
@pytest.mark.parametrize("mass,M5", [(1.0, 1.8), (0.3, 3.9)])
def test_cyclic_recurrence(env, ora, Ls, prec, mass, M5):
    """A^-1 and A^-dag where the boundary counts most: mass 1, and M5 = 3.9, where the recurrence's
    factor is 1 / 1.1 and its powers reach across the whole segment (one row of lanes, half a row
    or two)."""
    dwf, ctx = env
    P = dwf.PREC_NAMES[prec]
    dims = (4, 2, 2, 6)
    psi = mask(synth.gaussian_spinor(dims, Ls, 860 + Ls), dims, 0)
    lat = dwf.Lattice(ctx, dims, Ls, M5=M5, mass=mass)
    po = ora.params(dims, Ls, M5=M5, mass=mass)
    U = lat.pack_gauge(synth.random_links(dims, 0.5, 861), P)
    src = lat.pack(psi, dwf.KIND_EVEN, P)
    for dag in (False, True):
        dst = lat.empty(dwf.KIND_EVEN, P)
        dwf.dwf_dslash(ctx, lat.params(P), U, src, dst, dwf.OP_AINV, 0, dag)
        ref = mask(ora.fifth(po, psi, "Ainv" + ("dag" if dag else "")), dims, 0)
        err = rel_err(lat.unpack_np(dst, dwf.KIND_EVEN, P), ref)
        assert err < PREC_TOL[prec], (dag, err)


@pytest.mark.parametrize("dims,Ls", [((4, 2, 6, 2), 2), ((4, 2, 6, 2), 7), ((4, 2, 6, 2), 16), ((8, 8, 8, 10), 14)])
@pytest.mark.parametrize("prec", ["fp64", "fp32", "fp16", "bf16"])
@pytest.mark.parametrize("kind", ["shamir", "moebius", "sdep"])
def test_full_operator_and_input_factor(env, ora, dims, Ls, prec, kind):
    """D and D^dag with A applied to the hop's axpy operand (both chiralities' boundaries, odd and
    smallest extents, coefficients per slice), and H F and M_prec with the input factor in a pass of
    its own (FP64, FP32, the last lattice) or in the hop (16-bit, and the small ones)."""
    dwf, ctx = env
    P = dwf.PREC_NAMES[prec]
    kw, okw = {}, {}
    if kind == "moebius":
        kw = okw = {"b": 1.5, "c": 0.5}
    elif kind == "sdep":
        w = 1.5 + 0.5 * np.sin(np.arange(Ls))
        kw = {"b_s": (w + 1) / 2, "c_s": (w - 1) / 2}
        okw = {"bs": kw["b_s"], "cs": kw["c_s"]}
    U = synth.random_links(dims, 0.5, 870)
    psi = synth.gaussian_spinor(dims, Ls, 871 + Ls)
    lat = dwf.Lattice(ctx, dims, Ls, mass=0.2, tbc=1, **kw)
    po = ora.params(dims, Ls, mass=0.2, tbc=1, **okw)
    Ug, p = lat.pack_gauge(U, P), lat.params(P)
    src = lat.pack(psi, dwf.KIND_FULL, P)
    for dag in (False, True):
        dst = lat.empty(dwf.KIND_FULL, P)
        dwf.mobius_dslash(ctx, p, Ug, src, dst, dwf.OP_FULL, 0, dag)
        err = rel_err(lat.unpack_np(dst, dwf.KIND_FULL, P), ora.dwf(po, U, psi, dagger=dag))
        assert err < PREC_TOL[prec], ("D", dag, err)
    psio = mask(psi, dims, 1)
    srco = lat.pack(psio, dwf.KIND_ODD, P)
    out = lat.empty(dwf.KIND_ODD, P)
    dwf.mobius_dslash(ctx, p, Ug, srco, out, dwf.OP_MPREC, 1, False)
    err = rel_err(lat.unpack_np(out, dwf.KIND_ODD, P), ora.mprec(po, U, psio))
    assert err < PREC_TOL[prec], ("M", err)
    dwf.mobius_dslash(ctx, p, Ug, srco, out, dwf.OP_HOP, 0, False)
    ref = ora.hop5(po, U, ora.fifth(po, psio, "F"), out_parity=0)
    err = rel_err(lat.unpack_np(out, dwf.KIND_EVEN, P), ref)
    assert err < PREC_TOL[prec], ("HF", err)


@pytest.mark.parametrize("Ls", [2, 15, 16, 17, 33])
@pytest.mark.parametrize("prec", ["fp64", "fp32", "fp16", "bf16"])
def test_full_field_tiles(env, Ls, prec):
    """Full fields are packed and unpacked in tiles of sites and 16 slices; a full pack holds bit for bit
    what packing the even and odd halves (one thread per 5D site) gives, and unpacks to the same
    values as the two halves."""
    import torch
    dwf, ctx = env
    P = dwf.PREC_NAMES[prec]
    for dims in ((2, 2, 2, 2), (6, 4, 2, 10)):
        lat = dwf.Lattice(ctx, dims, Ls)
        psi = synth.gaussian_spinor(dims, Ls, 880 + Ls)
        psi[:, 0, 0, 0, 1] = 0.0  # (an FP16 site whose norm is that of zeros)
        full, halves = lat.zeros(dwf.KIND_FULL, P), [lat.zeros(k, P) for k in (dwf.KIND_EVEN, dwf.KIND_ODD)]
        src = lat.to_device(psi)
        dwf.dwf_pack(ctx, lat.params(P), dwf.KIND_FULL, P, src, full)
        for k, h in zip((dwf.KIND_EVEN, dwf.KIND_ODD), halves):
            dwf.dwf_pack(ctx, lat.params(P), k, P, src, h)
        assert torch.equal(full, torch.cat(halves))
        both = lat.unpack(halves[0], dwf.KIND_EVEN, P) + lat.unpack(halves[1], dwf.KIND_ODD, P)
        assert torch.equal(lat.unpack(full, dwf.KIND_FULL, P), both)


@pytest.mark.parametrize("Ls", [2, 3, 8, 9, 12, 13, 16, 17, 24, 31, 32, 33])
@pytest.mark.parametrize("prec", ["fp64", "fp32", "fp16", "bf16"])
def test_site_local_dense_products(env, ora, Ls, prec):
    """A^-1 and A^-dag with coefficients per slice (no recurrence at any extent): the matrix-core tiles
    at the edges of their extents (steps of 4 slices, 16 output slices, rows of 16 and 32 exchanged), the
    last one-lane-per-slice extent, and fewer sites than one workgroup or a part of a second one."""
    dwf, ctx = env
    P = dwf.PREC_NAMES[prec]
    w = 1.5 + 0.5 * np.sin(np.arange(Ls))
    b_s, c_s = (w + 1) / 2, (w - 1) / 2
    for dims in ((2, 2, 2, 2), (4, 6, 2, 6)):
        psi = mask(synth.gaussian_spinor(dims, Ls, 890 + Ls), dims, 0)
        lat = dwf.Lattice(ctx, dims, Ls, mass=0.3, b_s=b_s, c_s=c_s)
        po = ora.params(dims, Ls, mass=0.3, bs=b_s, cs=c_s)
        U = lat.pack_gauge(synth.random_links(dims, 0.5, 891), P)
        src = lat.pack(psi, dwf.KIND_EVEN, P)
        for dag in (False, True):
            dst = lat.empty(dwf.KIND_EVEN, P)
            dwf.mobius_dslash(ctx, lat.params(P), U, src, dst, dwf.OP_AINV, 0, dag)
            ref = mask(ora.fifth(po, psi, "Ainv" + ("dag" if dag else "")), dims, 0)
            err = rel_err(lat.unpack_np(dst, dwf.KIND_EVEN, P), ref)
            assert err < PREC_TOL[prec], (dims, dag, err)


@pytest.mark.parametrize("dims,Ls", [((2, 2, 2, 2), 2), ((4, 2, 6, 2), 7), ((2, 4, 2, 6), 12), ((2, 2, 6, 2), 16),
                                     ((2, 4, 2, 2), 32), ((2, 2, 2, 4), 63), ((2, 2, 2, 4), 64), ((2, 2, 2, 4), 65),
                                     ((8, 8, 8, 8), 16), ((8, 8, 8, 12), 16), ((8, 8, 8, 16), 16), ((8, 8, 8, 12), 17)])
@pytest.mark.parametrize("prec", ["fp64", "fp32", "fp16", "bf16"])
@pytest.mark.parametrize("b,c", [(1.0, 0.0), (1.5, 0.5)])
def test_small_field_hop(env, dims, Ls, prec, b, c):
    """Hop, M_prec and adjoints of fields below the size at which the directions stop being spread over
    the waves (32768 5D sites in 16 bit, 49152 in FP64, 65536 in FP32; extents to 64), at the
    limits and beyond: the default shape against an explicit one, which takes the general kernel."""
    dwf, ctx = env
    P = dwf.PREC_NAMES[prec]
    lat = dwf.Lattice(ctx, dims, Ls, mass=0.2, b=b, c=c, tbc=1)
    Ug, p = lat.pack_gauge(synth.random_links(dims, 0.5, 900), P), lat.params(P)
    src = lat.pack(synth.gaussian_spinor(dims, Ls, 901 + Ls), dwf.KIND_ODD, P)

    def results():
        out = []
        for op, par, kind in ((dwf.OP_HOP, 0, dwf.KIND_EVEN), (dwf.OP_MPREC, 1, dwf.KIND_ODD)):
            for dag in (False, True):
                dst = lat.empty(kind, P)
                dwf.mobius_dslash(ctx, p, Ug, src, dst, op, par, dag)
                out.append(lat.unpack_np(dst, kind, P))
        return out

    default = results()
    dwf.dwf_tune_set(ctx, P, Ls, min(16, max(1, 128 // Ls)), 1)
    try:
        explicit = results()
    finally:
        dwf.dwf_tune_set(ctx, P, Ls, 0, 0)
    for i, (a, e) in enumerate(zip(default, explicit)):
        assert rel_err(a, e) < PREC_TOL[prec], i


def bf16_rounded(a):
    """complex128 with both parts rounded to bf16"""
    import torch
    t = torch.from_numpy(np.ascontiguousarray(a).view(np.float64)).to(torch.bfloat16).to(torch.float64)
    return t.numpy().view(np.complex128)


@pytest.mark.parametrize("Ls", [8, 12, 16])
@pytest.mark.parametrize("kind", ["moebius", "sdep"])
@pytest.mark.parametrize("shape", ["default", "explicit"])
def test_bf16_moebius_stores_the_even_field_before_the_input_factor(env, ora, Ls, kind, shape):
    """M_prec in bf16 stores A^-1 H F psi on the even sites, and its second hop applies F.  On inputs of
    bf16 values the result is, up to FP32 arithmetic, the FP64 composition with that field rounded to
    bf16, rounded once more: an FP32 sum falls on the other side of a rounding boundary (relative error
    of a few 2^-24 against a spacing of 2^-8) once in some 10^4 components, and each of the about 10^3
    even components an output depends on moves it by a tenth of its spacing or less, so that about one
    output in a hundred may differ.  A field stored after F has other roundings in every component."""
    dwf, ctx = env
    dims = (4, 4, 2, 6)
    kw, okw = {"b": 1.5, "c": 0.5}, {"b": 1.5, "c": 0.5}
    if kind == "sdep":
        w = 1.5 + 0.5 * np.sin(np.arange(Ls))
        kw = {"b_s": (w + 1) / 2, "c_s": (w - 1) / 2}
        okw = {"bs": kw["b_s"], "cs": kw["c_s"]}
    U = bf16_rounded(synth.random_links(dims, 0.5, 910))
    psi = bf16_rounded(mask(synth.gaussian_spinor(dims, Ls, 911 + Ls), dims, 1))
    lat = dwf.Lattice(ctx, dims, Ls, mass=0.2, tbc=1, **kw)
    po = ora.params(dims, Ls, mass=0.2, tbc=1, **okw)
    Ug, p = lat.pack_gauge(U, dwf.BF16), lat.params(dwf.BF16)
    src, out = lat.pack(psi, dwf.KIND_ODD, dwf.BF16), lat.empty(dwf.KIND_ODD, dwf.BF16)
    if shape == "explicit":
        dwf.dwf_tune_set(ctx, dwf.BF16, Ls, 128 // Ls, 1)
    try:
        dwf.mobius_dslash(ctx, p, Ug, src, out, dwf.OP_MPREC, 1, False)
    finally:
        dwf.dwf_tune_set(ctx, dwf.BF16, Ls, 0, 0)
    got = lat.unpack_np(out, dwf.KIND_ODD, dwf.BF16)
    even = ora.fifth(po, ora.hop5(po, U, ora.fifth(po, psi, "F"), out_parity=0), "Ainv")
    second = ora.hop5(po, U, ora.fifth(po, bf16_rounded(even), "F"), out_parity=1)
    ref = psi - 0.25 * mask(ora.fifth(po, second, "Ainv"), dims, 1)
    other = (got != bf16_rounded(ref))[mask(np.ones_like(psi), dims, 1) != 0]
    assert other.mean() < 0.05


def recurrence(v, dtype, a, m, alpha, wide):
    """y_s = v_s / alpha + a y_{s-1} with y_{-1} = -m y_{Ls-1} along axis 0, in dtype: a doubling scan with
    zero start and the boundary in closed form, every step one fused multiply-add (formed in wide)"""
    def fma(x, y, z):
        return (wide(x) * y.astype(wide) + z.astype(wide)).astype(dtype)

    L = v.shape[0]
    f = dtype
    ap, av = f(a), f(a)
    y = (f(1 / alpha) * v).astype(dtype)
    off = 1
    while off < L:
        y = np.concatenate([y[:off], fma(ap, y[:-off], y[off:])])
        ap = f(ap * ap)
        off *= 2
    w = f(-m / (1 + m * wide(a) ** L))
    return np.stack([fma(f(w * av ** f(s + 1)), y[L - 1], y[s]) for s in range(L)])


@pytest.mark.parametrize("Ls", [8, 16, 32])
@pytest.mark.parametrize("prec", ["fp32", "fp64"])
@pytest.mark.parametrize("b,c", [(1.0, 0.0), (1.5, 0.5)])
@pytest.mark.parametrize("m", [0.01, 0.4])
def test_recurrence_is_as_accurate_as_its_steps(env, Ls, prec, b, c, m):
    """A^-1 in recurrence form is no further from the exact result (root mean square) than the scan with
    zero start and closed boundary evaluated on the host in the same precision.  Rounding is the same
    random process on both sides (10^5 components: 0.3 % of scatter), so the bound is 1.02 times."""
    dwf, ctx = env
    P = dwf.PREC_NAMES[prec]
    dtype, wide = (np.float32, np.float64) if prec == "fp32" else (np.float64, np.longdouble)
    dims = (4, 4, 4, 6)
    psi = mask(synth.gaussian_spinor(dims, Ls, 920 + Ls), dims, 1)
    lat = dwf.Lattice(ctx, dims, Ls, mass=m, b=b, c=c)
    Ug, p = lat.pack_gauge(synth.random_links(dims, 0.5, 921), P), lat.params(P)
    src, out = lat.pack(psi, dwf.KIND_ODD, P), lat.empty(dwf.KIND_ODD, P)
    v = lat.unpack_np(src, dwf.KIND_ODD, P)  # (as stored)
    dwf.mobius_dslash(ctx, p, Ug, src, out, dwf.OP_AINV, 1, False)
    got = lat.unpack_np(out, dwf.KIND_ODD, P)
    d = 4.0 - 1.8
    alpha, beta = b * d + 1.0, c * d - 1.0
    a = -np.longdouble(beta) / np.longdouble(alpha)

    def parts(x, flip):  # one chirality as real numbers, slices in the recurrence's direction
        r = np.ascontiguousarray(x[..., 2:, :] if flip else x[..., :2, :]).view(np.float64)
        return r[::-1] if flip else r

    err = {"gpu": 0.0, "host": 0.0}
    for flip in (False, True):
        u = parts(v, flip)
        exact = recurrence(u.astype(np.longdouble), np.longdouble, a, m, np.longdouble(alpha), np.longdouble)
        host = recurrence(u.astype(dtype), dtype, a, m, alpha, wide)
        err["host"] += float(np.sum((host.astype(np.longdouble) - exact) ** 2))
        err["gpu"] += float(np.sum((parts(got, flip).astype(np.longdouble) - exact) ** 2))
    assert err["gpu"] <= 1.02 ** 2 * err["host"], (err["gpu"] / err["host"]) ** 0.5


@pytest.mark.parametrize("prec", ["fp64", "fp32"])
@pytest.mark.parametrize("Ls", [12, 16])
def test_moebius_hop_and_operator_use_no_workspace(env, prec, Ls):
    """H F and D of the Moebius operator need the context's tables only: with the workspace released
    they can be captured in a graph (nothing is allocated), and the graph holds no pointer into a
    workspace that a later call may move: its replays, with the workspace in use between them, give
    the eager results bit for bit.  Above and below 65536 5D sites."""
    import torch
    dwf, _ = env
    P = dwf.PREC_NAMES[prec]
    stream = torch.cuda.Stream()
    with torch.cuda.stream(stream):
        ctx = dwf.Context(stream.cuda_stream)
        for dims in ((4, 4, 4, 6), (8, 8, 8, 24)):
            lat = dwf.Lattice(ctx, dims, Ls, mass=0.2, b=1.5, c=0.5)
            Ug, p = lat.pack_gauge(synth.random_links(dims, 0.5, 930), P), lat.params(P)
            src = lat.pack(synth.gaussian_spinor(dims, Ls, 931), dwf.KIND_FULL, P)
            odd = lat.pack(synth.gaussian_spinor(dims, Ls, 932), dwf.KIND_ODD, P)
            full, even, other = lat.zeros(dwf.KIND_FULL, P), lat.zeros(dwf.KIND_EVEN, P), lat.zeros(dwf.KIND_ODD, P)

            def apply():
                dwf.mobius_dslash(ctx, p, Ug, odd, even, dwf.OP_HOP, 0, False)
                dwf.mobius_dslash(ctx, p, Ug, src, full, dwf.OP_FULL, 0, False)

            apply()
            stream.synchronize()
            want = full.clone(), even.clone()
            ctx.release()
            graph = torch.cuda.CUDAGraph()
            with torch.cuda.graph(graph, stream=stream):
                apply()
            for _ in range(3):
                full.zero_()
                even.zero_()
                dwf.mobius_dslash(ctx, p, Ug, odd, other, dwf.OP_MPREC, 1, True)
                graph.replay()
                stream.synchronize()
                assert torch.equal(full, want[0]) and torch.equal(even, want[1])
                ctx.release()
        ctx.close()


@pytest.mark.parametrize("prec", ["fp64", "fp32"])
@pytest.mark.parametrize("dag", [False, True])
def test_operator_coefficients_are_rounded_once(env, prec, dag):
    """D with coefficients per slice on zero links is A = alpha_s + beta_s S~.  On a field of one slice
    the result's slices are that slice times alpha_s, beta_s (-m beta_s across the boundary); the best
    fit of the factor averages the products' own rounding away and leaves the factor's: at most half a
    unit, 2^-24 (2^-53) relative, and as much again where -m multiplies it.  (10^4 components: the
    average's own scatter is a hundredth of a unit.)"""
    dwf, ctx = env
    P = dwf.PREC_NAMES[prec]
    dims, Ls, m, d = (4, 4, 4, 6), 7, 0.3, 4.0 - 1.8
    half = 2.0 ** (-53 if prec == "fp64" else -24)
    w = 1.5 + 0.5 * np.sin(np.arange(Ls))
    b_s, c_s = (w + 1) / 2, (w - 1) / 2
    lat = dwf.Lattice(ctx, dims, Ls, mass=m, b_s=b_s, c_s=c_s)
    Ug, p = lat.pack_gauge(np.zeros_like(synth.random_links(dims, 0.5, 940)), P), lat.params(P)
    for s in range(Ls):
        psi = np.zeros_like(synth.gaussian_spinor(dims, Ls, 941))
        psi[s] = synth.gaussian_spinor(dims, Ls, 941 + s)[s]
        src, dst = lat.pack(psi, dwf.KIND_FULL, P), lat.empty(dwf.KIND_FULL, P)
        x = lat.unpack_np(src, dwf.KIND_FULL, P)[s].astype(np.clongdouble)
        dwf.mobius_dslash(ctx, p, Ug, src, dst, dwf.OP_FULL, 0, dag)
        got = lat.unpack_np(dst, dwf.KIND_FULL, P).astype(np.clongdouble)
        for ch, spins in ((0, slice(0, 2)), (1, slice(2, 4))):
            n = s + (1 if ch == 0 else -1) * (-1 if dag else 1)  # the slice that reads slice s
            wrap = n < 0 or n >= Ls
            n %= Ls
            row = s if dag else n
            want = {s: b_s[s] * d + 1, n: (c_s[row] * d - 1) * (-m if wrap else 1)}  # (formed in FP64)
            for t, f in want.items():
                xs = x[..., spins, :]
                fit = np.sum((got[t][..., spins, :] * xs.conj()).real) / np.sum(np.abs(xs) ** 2)
                assert abs(fit / np.longdouble(f) - 1) < half * (2.1 if wrap and t == n else 1.1), (s, ch, t)


@pytest.mark.parametrize("Ls", [8, 16, 32])
@pytest.mark.parametrize("b,c", [(1.5, 0.5), (1.6, 0.6)])
def test_moebius_mprec_with_the_factor_in_the_epilogue(env, Ls, b, c):
    """M_prec in FP32 with F A^-1 as the first hop's epilogue is no further from the exact result (FP64 on the
    same stored values) than the composition with F in the second hop: H F, A^-1, H F, A^-1 as calls of
    their own, the axpy in FP64.  (10^6 components: the ratio of the two errors scatters by 0.1 %.)"""
    dwf, ctx = env
    dims = (8, 8, 8, 12)
    lats = dwf.Lattice(ctx, dims, Ls, mass=0.05, b=b, c=c)
    U = synth.random_links(dims, 0.5, 950).astype(np.complex64).astype(np.complex128)
    res = {}
    for prec in ("fp64", "fp32"):
        P = dwf.PREC_NAMES[prec]
        Ug, p = lats.pack_gauge(U, P), lats.params(P)
        psi = mask(synth.gaussian_spinor(dims, Ls, 951), dims, 1).astype(np.complex64).astype(np.complex128)
        src = lats.pack(psi, dwf.KIND_ODD, P)
        out, even = lats.empty(dwf.KIND_ODD, P), lats.empty(dwf.KIND_EVEN, P)
        even2, odd, odd2 = lats.empty(dwf.KIND_EVEN, P), lats.empty(dwf.KIND_ODD, P), lats.empty(dwf.KIND_ODD, P)
        dwf.dwf_tune_set(ctx, P, Ls, 128 // Ls, 1)  # (the general kernel on both sides)
        try:
            dwf.mobius_dslash(ctx, p, Ug, src, out, dwf.OP_MPREC, 1, False)
            dwf.mobius_dslash(ctx, p, Ug, src, even, dwf.OP_HOP, 0, False)
            dwf.mobius_dslash(ctx, p, Ug, even, even2, dwf.OP_AINV, 0, False)
            dwf.mobius_dslash(ctx, p, Ug, even2, odd, dwf.OP_HOP, 1, False)
            dwf.mobius_dslash(ctx, p, Ug, odd, odd2, dwf.OP_AINV, 1, False)
        finally:
            dwf.dwf_tune_set(ctx, P, Ls, 0, 0)
        res[prec] = lats.unpack_np(out, dwf.KIND_ODD, P), psi - 0.25 * lats.unpack_np(odd2, dwf.KIND_ODD, P)
    exact = res["fp64"][0]
    err = [np.linalg.norm(r - exact) for r in res["fp32"]]
    assert err[0] <= 1.01 * err[1], err[0] / err[1]


@pytest.mark.parametrize("prec", ["fp64", "fp32", "bf16"])
@pytest.mark.parametrize("shape", ["default", "explicit"])
def test_5d_hop_reads_neighbouring_slices_only(env, prec, shape):
    """K takes a site's own 4D parity from slices s - 1 and s + 1, never from s: an infinite component in
    one slice of one site leaves that slice of that site as it is without it."""
    dwf, ctx = env
    P = dwf.PREC_NAMES[prec]
    dims, Ls, s = (4, 4, 2, 6), 8, 3
    lat = dwf.Lattice(ctx, dims, Ls, mass=0.2)
    Ug, p = lat.pack_gauge(synth.random_links(dims, 0.5, 960), P), lat.params(P)
    psi = synth.gaussian_spinor(dims, Ls, 961)
    if shape == "explicit":
        dwf.dwf_tune_set(ctx, P, Ls, 16, 1)
    try:
        for dag in (False, True):
            out = []
            for v in (0.0, np.inf):
                psi[s, 2, 1, 1, 3] = v  # one spinor
                src, dst = lat.pack(psi, dwf.KIND_FULL, P), lat.empty(dwf.KIND_FULL, P)
                dwf.dwf_dslash_5d(ctx, p, Ug, src, dst, dwf.OP5_HOP, dag)
                out.append(lat.unpack_np(dst, dwf.KIND_FULL, P)[s, 2, 1, 1, 3])
            assert np.isfinite(out[0]).all() and np.array_equal(out[0], out[1]), dag
    finally:
        dwf.dwf_tune_set(ctx, P, Ls, 0, 0)


@pytest.mark.parametrize("prec", ["fp64", "fp32", "fp16", "bf16"])
def test_timer_names_the_small_field_kernel(env, prec):
    """The report names the kernel that ran: hop_split_kernel at the default shape of a small field,
    hop_kernel with a shape set explicitly and on a larger field."""
    dwf, ctx = env
    P, Ls, tag = dwf.PREC_NAMES[prec], 16, {"fp64": "P64", "fp32": "P32", "fp16": "P16", "bf16": "PB16"}[prec]

    def names(dims):
        lat = dwf.Lattice(ctx, dims, Ls, mass=0.2)
        Ug, p = lat.pack_gauge(synth.random_links(dims, 0.5, 970), P), lat.params(P)
        src, dst = lat.pack(synth.gaussian_spinor(dims, Ls, 971), dwf.KIND_ODD, P), lat.empty(dwf.KIND_ODD, P)
        dwf.dwf_timing_report(ctx)
        dwf.dwf_timing_enable(ctx, True)
        try:
            dwf.dwf_dslash(ctx, p, Ug, src, dst, dwf.OP_MPREC, 1, False)
            return dwf.dwf_timing_report(ctx)
        finally:
            dwf.dwf_timing_enable(ctx, False)

    small = names((4, 4, 4, 4))
    assert set(small) == {f"hop_split_kernel<dwf::{tag}, 16, false, false, 2, false>"}
    assert next(iter(small.values()))["launches"] == 2
    general = {f"hop_kernel<dwf::{tag}, 16, 1, false, false, 2, {'false' if prec == 'fp16' else 'true'}, false, false>"}
    assert set(names((8, 8, 8, 24))) == general
    dwf.dwf_tune_set(ctx, P, Ls, *dwf.dwf_tune_get(ctx, P, Ls))
    try:
        assert set(names((4, 4, 4, 4))) == general
    finally:
        dwf.dwf_tune_set(ctx, P, Ls, 0, 0)


@pytest.mark.parametrize("Ls,spb,ns", [(7, 18, 1), (16, 8, 1), (16, 8, 2), (32, 4, 4)])
@pytest.mark.parametrize("prec", ["fp64", "fp32", "bf16"])
@pytest.mark.parametrize("kind", ["shamir", "moebius", "sdep"])
def test_full_operator_in_the_general_kernel(env, ora, Ls, spb, ns, prec, kind):
    """D and D^dag with A on the axpy operand in the kernel that larger fields take, one and several
    slices per thread, against the oracle."""
    dwf, ctx = env
    P, dims = dwf.PREC_NAMES[prec], (4, 2, 6, 4)
    kw, okw = {}, {}
    if kind == "moebius":
        kw = okw = {"b": 1.5, "c": 0.5}
    elif kind == "sdep":
        w = 1.5 + 0.5 * np.sin(np.arange(Ls))
        kw = {"b_s": (w + 1) / 2, "c_s": (w - 1) / 2}
        okw = {"bs": kw["b_s"], "cs": kw["c_s"]}
    U = synth.random_links(dims, 0.5, 980)
    psi = synth.gaussian_spinor(dims, Ls, 981 + Ls)
    lat = dwf.Lattice(ctx, dims, Ls, mass=0.2, tbc=1, **kw)
    po = ora.params(dims, Ls, mass=0.2, tbc=1, **okw)
    Ug, p, src = lat.pack_gauge(U, P), lat.params(P), lat.pack(psi, dwf.KIND_FULL, P)
    dwf.dwf_tune_set(ctx, P, Ls, spb, ns)
    try:
        for dag in (False, True):
            dst = lat.empty(dwf.KIND_FULL, P)
            dwf.mobius_dslash(ctx, p, Ug, src, dst, dwf.OP_FULL, 0, dag)
            err = rel_err(lat.unpack_np(dst, dwf.KIND_FULL, P), ora.dwf(po, U, psi, dagger=dag))
            assert err < PREC_TOL[prec], (dag, err)
    finally:
        dwf.dwf_tune_set(ctx, P, Ls, 0, 0)


def test_traversal_tile_in_the_general_kernel(env, ora):
    """Every traversal tile gives bit-identical M_prec and M_prec^dag that agree with the oracle, in the
    kernel that reads the order (a shape set explicitly: small fields at the default shape do not)."""
    dwf, ctx = env
    P, dims, Ls = dwf.FP32, (12, 4, 6, 8), 8
    U = synth.random_links(dims, 0.5, 990)
    psio = mask(synth.gaussian_spinor(dims, Ls, 991), dims, 1)
    lat = dwf.Lattice(ctx, dims, Ls, mass=0.05, b=1.5, c=0.5, tbc=1)
    Ug, src = lat.pack_gauge(U, P), lat.pack(psio, dwf.KIND_ODD, P)
    po = ora.params(dims, Ls, mass=0.05, b=1.5, c=0.5, tbc=1)
    dwf.dwf_tune_set(ctx, P, Ls, *dwf.dwf_tune_get(ctx, P, Ls))
    try:
        first = {}
        for tile in [(0, 0, 0), (2, 2, 2), (12, 4, 6), (4, 2, 3), (6, 4, 2), (3, 1, 1)]:
            dwf.dwf_tune_tile(ctx, dims, tile, 1)
            for dag in (False, True):
                dst = lat.empty(dwf.KIND_ODD, P)
                dwf.mobius_dslash(ctx, lat.params(P), Ug, src, dst, dwf.OP_MPREC, 1, dag)
                got = lat.unpack_np(dst, dwf.KIND_ODD, P)
                if dag not in first:
                    first[dag] = got
                    assert rel_err(got, ora.mprec(po, U, psio, dagger=dag)) < PREC_TOL["fp32"]
                assert np.array_equal(got, first[dag]), (tile, dag)
    finally:
        dwf.dwf_tune_tile(ctx, dims, (0, 0, 0), 1)
        dwf.dwf_tune_set(ctx, P, Ls, 0, 0)


def test_autotuner_keeps_the_default_where_it_is_faster(env, tmp_path, monkeypatch):
    """The search times the library's own choice beside the explicit shapes and installs and caches it where
    it wins: on a small field it is a kernel that no explicit shape selects."""
    from paper_1111_5059_amd import autotune
    dwf, ctx = env
    dims, Ls, P = (4, 4, 4, 4), 16, dwf.FP32
    lat = dwf.Lattice(ctx, dims, Ls, mass=0.05)
    U64 = lat.pack_gauge(synth.random_links(dims, 0.5, 995))
    cache = str(tmp_path / "tune.json")
    monkeypatch.setattr(autotune, "candidates", lambda P, Ls: [{"spb": 1, "ns": 1, "xcd": 0, "ll": 0}])
    try:
        best, ms, table = autotune.tune_hop(lat, U64, "fp32", reps=20, cache=cache)
        assert best == autotune.DEFAULT_SHAPE and len(table) == 2 and ms == min(r["ms"] for r in table)
        dwf.dwf_tune_set(ctx, P, Ls, 1, 1)
        assert autotune.load(lat, "fp32", cache) == dict(best, ms=ms)
        src, dst = lat.zeros(dwf.KIND_ODD, P), lat.empty(dwf.KIND_ODD, P)
        Ug = lat.pack_gauge(synth.random_links(dims, 0.5, 995), P)
        dwf.dwf_timing_report(ctx)
        dwf.dwf_timing_enable(ctx, True)
        dwf.dwf_dslash(ctx, lat.params(P), Ug, src, dst, dwf.OP_MPREC, 1, False)
        assert all(k.startswith("hop_split_kernel<") for k in dwf.dwf_timing_report(ctx))
    finally:
        dwf.dwf_timing_enable(ctx, False)
        dwf.dwf_tune_set(ctx, P, Ls, 0, 0)


BLOCKING_SOLVE = """
import ctypes, time
assert ctypes.CDLL("libamdhip64.so").hipSetDeviceFlags(4) == 0  # hipDeviceScheduleBlockingSync
import torch, paper_1111_5059_amd as dwf
ctx = dwf.Context()
lat = dwf.Lattice(ctx, (24, 24, 24, 24), 16, mass=0.01)
b, x = lat.empty(dwf.KIND_FULL), lat.zeros(dwf.KIND_FULL)
b.view(torch.float64).normal_()
U = lat.empty(dwf.KIND_GAUGE)
U.view(torch.float64).normal_(std=0.3)
dwf.cg_ne(ctx, lat.params(), U, b, x, tol=1e-14, maxit=2)
x.zero_()
torch.cuda.synchronize()
c, w = time.process_time(), time.perf_counter()
dwf.cg_ne(ctx, lat.params(), U, b, x, tol=1e-14, maxit=100)
print("share", (time.process_time() - c) / (time.perf_counter() - w))
"""


def test_blocking_device_schedule_is_kept():
    """A program that set its device to blocking waits is not kept busy by a solve whose iterations take
    milliseconds (a wait that spins uses a whole core, and the threads of the runtime a little more)."""
    import os
    import subprocess
    import sys
    root = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
    r = subprocess.run([sys.executable, "-c", BLOCKING_SOLVE], capture_output=True, text=True, timeout=100, cwd=root,
                       env=dict(os.environ, PYTHONPATH=root))
    assert r.returncode == 0, r.stderr[-2000:]
    assert float(r.stdout.split("share")[1]) < 0.6, r.stdout
