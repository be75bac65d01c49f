"""Performance cases: the calls a user of the imager makes, over the range of sizes it is used at.

Every case is a plain dict with a `kind`:

* apply      Phi then Phi^H with one exact G (stored taps in a type, with or without factor records, or the
             records alone)
* batch      the same for several channels bound into one Batch
* build      build_G: the sparse rows, their transposed copy and the block table
* solve      ||Phi||^2 by power iteration, then the primal-dual reconstruction
* train      one minibatch step of the surrogate network: gradients and an Adam step
* infer      the network's rows for a batch of visibilities
* surrogate  Phi then Phi^H with network rows and exact fallback rows

`prepare` makes a case's inputs from a seed, `run` is one pass through the public entry points, `exact` is the
same result in FP64 from the definitions, and `work` the bytes and operations one pass cannot do without.

Geometry: field of view 2 degrees, L = 2 sin(1 degree); w is drawn from [0, w_top) with w_top set by the largest
kernel support S in cells, w_top = (S - 4) / (4 L^2).
"""
from __future__ import annotations

import math

import numpy as np
import torch

import paper_1307_3424_amd as wp

L = 2.0 * math.sin(math.radians(1.0))
W = 4                                                 # Kaiser-Bessel support in cells
BETA = math.pi * math.sqrt((W / 2.0) ** 2 * 1.5 ** 2 - 0.8)
TAPS = {"c64": wp.WP_TAPS_C64, "bf16": wp.WP_TAPS_BF16, "i16": wp.WP_TAPS_I16}
H, BOX, NOUT = 256, 32, 2048                          # the surrogate network
TOL = 1e-3


# ------------------------------------------------------------------------------------------------ cases

def listed():
    return [
        # the tiny form: 64 pixels, chirp over half the grid, a few hundred baselines; a call is launches and latency
        dict(name="apply-tiny-64", kind="apply", N=64, M=820, S=0, E=0.99, taps="c64", form="stored", order="caller"),
        # the plain form: one snapshot at 256 pixels, as an iterative solver calls it
        dict(name="apply-plain-256", kind="apply", N=256, M=32768, S=32, E=0.99, taps="c64", form="stored",
             order="caller"),
        # the exact operator as a long reconstruction keeps it: taps, transposed copy and factor records, sorted vectors
        dict(name="apply-exact-1024", kind="apply", N=1024, M=400001, S=32, E=0.99, taps="c64", form="both",
             order="sorted"),
        # the precision form: wide kernels, bfloat16 taps
        dict(name="apply-bf16-1024", kind="apply", N=1024, M=131073, S=64, E=0.99, taps="bf16", form="stored",
             order="sorted"),
        # G kept as factor records alone, where stored taps would not fit
        dict(name="apply-records-2048", kind="apply", N=2048, M=600000, S=32, E=0.99, taps="c64", form="records",
             order="sorted"),
        # frequency channels of uneven size in one persistent launch
        dict(name="batch-512", kind="batch", N=512, Ms="50000,93001,171003,320000", S=32, E=0.99),
        # setting up a snapshot
        dict(name="build-256", kind="build", N=256, M=32768, S=32, E=0.99, taps="c64"),
        # setting up the largest image, in pieces of the visibility set
        dict(name="build-2048", kind="build", N=2048, M=65536, S=32, E=0.99, taps="c64"),
        # a whole reconstruction of the plain form: norm estimate and iterations
        dict(name="solve-256", kind="solve", N=256, M=32768, S=32, E=0.99, levels=4, power=20, iters=60),
        # one training step at the training batch
        dict(name="train-8192", kind="train", n=8192),
        # network rows for a ragged batch of visibilities
        dict(name="infer-10007", kind="infer", n=10007),
        # the learned operator with its fallback rows
        dict(name="surrogate-512", kind="surrogate", N=512, M=400001, S=32, E=0.99, fallback=0.38),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _taps_per_row(S, E):
    return {0.9: 0.15, 0.99: 0.22, 0.999: 0.4}[E] * max(S, 8) ** 2


def draw(rng):
    kind = rng.choice(["apply", "apply", "apply", "batch", "build", "build", "solve", "train", "infer", "surrogate"])
    E = rng.choice([0.9, 0.99, 0.99, 0.999])
    if kind == "apply":
        N = rng.choice([64, 128, 256, 512, 1024, 2048])
        S = rng.randint(8, 64 if N >= 256 else 32)
        M = _log_int(rng, 300, min(400001, 9e7 / _taps_per_row(S, E)))
        return dict(kind=kind, N=N, M=M, S=S, E=E, taps=rng.choice(["c64", "c64", "bf16", "i16"]),
                    form=rng.choice(["stored", "both", "records"]), order=rng.choice(["caller", "sorted"]))
    if kind == "batch":
        Ms = [_log_int(rng, 2000, 200000) for _ in range(rng.randint(2, 6))]
        return dict(kind=kind, N=rng.choice([128, 256, 512]), Ms=",".join(str(m) for m in Ms), S=rng.randint(8, 32),
                    E=rng.choice([0.9, 0.99]))
    if kind == "build":
        N = rng.choice([64, 128, 256, 512, 1024, 2048])
        return dict(kind=kind, N=N, M=_log_int(rng, 500, 60000), S=rng.randint(8, 32), E=E,
                    taps=rng.choice(["c64", "bf16", "i16"]))
    if kind == "solve":
        N = rng.choice([64, 128, 256, 512])
        return dict(kind=kind, N=N, M=_log_int(rng, 2000, 50000), S=rng.randint(8, 32), E=0.99,
                    levels=rng.choice([0, 2, 4]), power=rng.randint(5, 20), iters=rng.randint(10, 60))
    if kind == "train":
        return dict(kind=kind, n=64 * _log_int(rng, 1, 128))
    if kind == "infer":
        return dict(kind=kind, n=_log_int(rng, 1, 10007))
    return dict(kind=kind, N=rng.choice([128, 256, 512, 1024]), M=_log_int(rng, 3000, 400001), S=rng.randint(12, 32),
                E=0.99, fallback=rng.choice([0.0, 0.1, 0.38, 0.6]))


# ------------------------------------------------------------------------------------------------ inputs

def _gen(seed, stream):
    return np.random.default_rng([int(seed), stream])


def _dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def _w_top(case):
    return case["N"] / (2.0 * L * L) if case["S"] == 0 else (case["S"] - 4) / (4.0 * L * L)


def _uvw(N, M, w_top, seed, stream, uniform=False):
    """(u, v) isotropic Gaussian of sigma 0.25 B cut at the band limit B = N / (2 L), or uniform; w uniform."""
    r = _gen(seed, stream)
    B = N / (2.0 * L)
    out = []
    for _ in range(2):
        if uniform:
            out.append(r.uniform(-B, B, M))
            continue
        a = r.normal(0.0, 0.25 * B, M)
        while (bad := np.abs(a) >= B).any():
            a[bad] = r.normal(0.0, 0.25 * B, int(bad.sum()))
        out.append(a)
    out.append(r.uniform(0.0, w_top, M))
    return out


def _uvw_cells(N, M, w_top, seed):
    """As _uvw, every seed with the same w and offsets within a cell (so the same number of taps), the cells and
    the order of the visibilities its own."""
    fixed, r = _gen(0, 6), _gen(seed, 7)
    off, w = fixed.uniform(0.0, 1.0, (2, M)), fixed.uniform(0.0, w_top, M)
    p = r.permutation(M)
    cell = np.floor(np.clip(r.normal(0.0, 0.25 * N, (2, M)), -N + 1, N - 2))
    u, v = (cell + off[:, p]) / (2.0 * L)
    return [u, v, w[p]]


def _sky(N, seed, stream):
    """33 Gaussian blobs and 67 point sources, log-normal amplitudes (float64 CUDA, N x N)."""
    r = _gen(seed, stream)
    p = torch.arange(N, dtype=torch.float64, device="cuda")
    cy, cx, s, a = (_dev(z) for z in (r.uniform(0, N, 33), r.uniform(0, N, 33), r.uniform(1, 4, 33),
                                      r.lognormal(0, 1, 33)))
    gy = torch.exp(-(p[:, None] - cy) ** 2 / (2 * s * s)) * a
    gx = torch.exp(-(p[:, None] - cx) ** 2 / (2 * s * s))
    img = gy @ gx.T
    at = _dev(r.integers(0, N * N, 67))
    return img.view(-1).index_add(0, at, _dev(r.lognormal(0, 1, 67))).view(N, N)


def _vis(M, seed, stream):
    r = _gen(seed, stream)
    return (r.normal(size=M) + 1j * r.normal(size=M)).astype(np.complex64)


def _net(seed):
    """Seeded parameters, every weight and bias uniform in +-1/sqrt(fan_in), in the packed order."""
    r = _gen(seed, 40)
    parts = []
    for n, k in ((H, 3), (H, H), (H, H), (NOUT, H)):
        parts += [r.uniform(-1, 1, n * k) / math.sqrt(k), r.uniform(-1, 1, n) / math.sqrt(k)]
    return np.concatenate(parts).astype(np.float32)


def _features(n, seed):
    return _gen(seed, 41).uniform(-1.0, 1.0, (n, 3)).astype(np.float32)


def _targets(n, seed):
    """A box of mostly empty cells, the others of order one, as sparsified rows divided by the output scale."""
    g = torch.Generator(device="cuda").manual_seed(int(seed) * 7919 + 42)
    t = torch.randn(n, BOX * BOX, 2, generator=g, device="cuda")
    keep = torch.rand(n, BOX * BOX, 1, generator=g, device="cuda") < 0.2
    return torch.where(keep, t * 1.3, torch.zeros((), device="cuda")).reshape(-1).contiguous()


def _channels(case):
    Ms = [int(m) for m in case["Ms"].split(",")]
    return [(M, _w_top(case) * (0.5 + 0.5 * c / max(1, len(Ms) - 1))) for c, M in enumerate(Ms)]


def _over_tol(case, seed):
    """Row errors as a check finds them: the stated fraction above the tolerance."""
    r = _gen(seed, 43)
    e = r.uniform(0.1, 0.99, case["M"]) * TOL
    e[r.uniform(size=case["M"]) < case["fallback"]] = 4 * TOL
    return e.astype(np.float32)


def _solve_data(case, seed):
    """Noisy data of a sky at 30 dB and the radius of its l2 ball, from the rows' whole windows in FP64."""
    N, M = case["N"], case["M"]
    u, v, w = _uvw(N, M, _w_top(case), seed, 1)
    X = _grid64(_sky(N, seed, 2).to(torch.complex128), N)
    y = torch.cat([_full_rows(b, X) for b in _blocks(case, u, v, w)])
    sig = 10.0 ** -1.5 * float(torch.sqrt((y.abs() ** 2).mean()))
    r = _gen(seed, 3)
    y = y + _dev(sig * (r.normal(size=M) + 1j * r.normal(size=M)) / math.sqrt(2.0))
    return (u, v, w), y.to(torch.complex64), math.sqrt(sig * sig * (M + 2 * math.sqrt(M)))


def _start(case, seed):
    return _gen(seed, 4).normal(size=case["N"] ** 2).astype(np.float32)


def prepare(case, seed):
    kind = case["kind"]
    st = dict(kind=kind, case=case)
    if kind in ("train", "infer"):
        n = case["n"]
        st["mlp"] = wp.Mlp(max_batch=max(64, (n + 63) // 64 * 64))
        st["mlp"].set_params(_net(seed), 5745.0, 100.0)
        st["feat"] = _dev(_features(n, seed).reshape(-1))
        if kind == "train":
            st["target"] = _targets(n, seed)
        return st
    N = case["N"]
    plan = st["plan"] = wp.Plan(N, L)
    if kind == "batch":
        Gs, xs = [], []
        for c, (M, w_top) in enumerate(_channels(case)):
            G = wp.build_G(plan, *(_dev(a) for a in _uvw(N, M, w_top, seed, 100 + c)), case["E"])
            G.order = wp.WP_ORDER_SORTED
            Gs.append(G)
            xs.append(_sky(N, seed, 200 + c).to(torch.complex64).reshape(-1))
        st["batch"] = wp.Batch(plan, Gs)
        _, st["y"], st["grids"] = st["batch"].new_buffers()
        st["x"] = torch.cat(xs)
        st["xa"] = torch.empty_like(st["x"])
        st["yin"] = _dev(_vis(st["batch"].M_total, seed, 5))
        return st
    if kind == "solve":
        (u, v, w), y, st["eps"] = _solve_data(case, seed)
        G = st["G"] = wp.build_G(plan, _dev(u), _dev(v), _dev(w), case["E"])
        G.order = wp.WP_ORDER_SORTED
        st["y"] = wp.to_sorted(G, y)
        st["x0"] = _dev(_start(case, seed))
        return st
    M = case["M"]
    if kind == "build":
        st["uvw"] = [_dev(a) for a in _uvw_cells(N, M, _w_top(case), seed)]
        return st
    uvw = [_dev(a) for a in _uvw(N, M, _w_top(case), seed, 1, uniform=case["S"] == 0)]
    st["x"] = _sky(N, seed, 2).to(torch.complex64).reshape(-1).contiguous()
    st["y"] = _dev(_vis(M, seed, 5))
    st["grid"] = plan.new_grid()
    if kind == "apply":
        form = case["form"]
        G = st["G"] = wp.build_G(plan, *uvw, case["E"], taps=TAPS[case["taps"]], transpose=form != "records",
                                 factors=form != "stored", stored=form != "records")
        if case["order"] == "sorted":
            G.order = wp.WP_ORDER_SORTED
        return st
    mlp = wp.Mlp(max_batch=8192)
    mlp.set_params(_net(seed), _w_top(case), wp.Mlp.output_scale(plan))
    sur = st["sur"] = wp.Surrogate(plan, mlp, *uvw, eps=_dev(_over_tol(case, seed)), tol=TOL)
    st["Gf"] = None
    if sur.Mf:
        st["Gf"] = wp.build_G(plan, *sur.fallback_coords(), case["E"], factors=True)
        st["Gf"].order = wp.WP_ORDER_SORTED
    return st


# ------------------------------------------------------------------------------------------------ one pass

def run(st):
    kind, case = st["kind"], st["case"]
    if kind == "apply":
        y = wp.apply_Phi(st["plan"], st["G"], st["x"], grid=st["grid"])
        x = wp.apply_PhiT(st["plan"], st["G"], st["y"], grid=st["grid"])
        return {"y": y, "x": x}
    if kind == "batch":
        y = st["batch"].apply_Phi(st["x"], st["y"], st["grids"])
        x = st["batch"].apply_PhiT(st["yin"], st["xa"], st["grids"])
        return {"y": y, "x": x}
    if kind == "build":
        G = wp.build_G(st["plan"], *st["uvw"], case["E"], taps=TAPS[case["taps"]])
        return {k: getattr(G, k) for k in ("rowptr", "col", "val", "perm", "tcolptr", "trow", "tval")}
    if kind == "solve":
        nu = wp.power_norm2(st["plan"], st["G"], st["x0"], case["power"])
        x = wp.solve(st["plan"], st["G"], st["y"], st["eps"], 1.05 * nu, case["iters"], case["levels"])
        return {"nu": nu, "x": x}
    if kind == "train":
        grads, loss = st["mlp"].gradients(st["feat"], st["target"])
        st["mlp"].adam_step(0.0)                     # the first rate of a warm-up: every pass trains the same weights
        return {"grads": grads, "loss": loss}
    if kind == "infer":
        return {"out": st["mlp"].forward(st["feat"])}
    y = st["sur"].apply_Phi(st["x"], grid=st["grid"], Gf=st["Gf"])
    x = st["sur"].apply_PhiT(st["y"], grid=st["grid"], Gf=st["Gf"])
    return {"y": y, "x": x}


# ------------------------------------------------------------------------------------------------ work

def work(case):
    """Both products read their operator once and their vectors once; network kinds: the layers' products."""
    kind = case["kind"]
    if kind in ("train", "infer"):
        n, per = case["n"], 2 * (3 * H + 2 * H * H + H * NOUT)
        if kind == "infer":
            return {"bytes": 4 * n * (3 + NOUT) + 2 * per, "flops": n * per}
        return {"bytes": 4 * n * (3 + NOUT) + 12 * per, "flops": 3 * n * per}
    N = case["N"]
    S = case["S"] or N
    nnz1 = _taps_per_row(S, case["E"])
    if kind == "batch":
        Ms = [M for M, _ in _channels(case)]
        taps = sum(Ms) * nnz1 * 0.6
        return {"bytes": 24 * taps + 16 * sum(Ms) + len(Ms) * 32 * N * N, "flops": 16 * taps}
    M = case["M"]
    taps = M * nnz1
    vec = 16 * M + 16 * N * N
    rec = M * (10.0 * S + 8)
    if kind == "apply":
        one = {"c64": 12, "bf16": 8, "i16": 8}[case["taps"]]
        deg = rec if case["form"] != "stored" else one * taps
        gat = rec if case["form"] == "records" else one * taps
        return {"bytes": deg + gat + vec, "flops": 16 * taps}
    if kind == "build":
        one = {"c64": 12, "bf16": 8, "i16": 8}[case["taps"]]
        Ng = 2 * N
        return {"bytes": 24 * M + 2 * one * taps + 12 * M + 8 * Ng * Ng,
                "flops": M * (5 * Ng * math.log2(Ng) + 32 * Ng)}
    if kind == "solve":
        n = case["power"] + case["iters"]
        return {"bytes": n * (24 * taps + vec), "flops": n * 16 * taps}
    net = M * (1 - case["fallback"])
    fb = M - net
    # output layer once per occupied cell (cells of the Gaussian's core), hidden layers read once per product
    cells = min(net, 2 * math.pi * (0.25 * N) ** 2 * math.log(1 + net / (2 * math.pi * (0.25 * N) ** 2)) + 1)
    return {"bytes": 2 * 2 * H * net + fb * (10.0 * S + 12 * nnz1) + vec,
            "flops": 2 * 2 * H * NOUT * cells * 2 + 16 * fb * nnz1}


# ------------------------------------------------------------------------------------------------ FP64 results

def _apod64(N):
    xi = (torch.arange(N, dtype=torch.float64, device="cuda") - N / 2) / (2 * N)
    s = torch.sqrt(BETA ** 2 - (math.pi * W * xi) ** 2)          # positive over |xi| <= 1/4
    g = W * torch.sinh(s) / s
    return 1.0 / (g[:, None] * g[None, :])


def _grid64(x, N):
    """F Z A x: centred transform of the apodised, zero-padded image (flat)."""
    z = torch.zeros(2 * N, 2 * N, dtype=torch.complex128, device="cuda")
    z[N // 2:N // 2 + N, N // 2:N // 2 + N] = x.view(N, N) * _apod64(N)
    return torch.fft.fftshift(torch.fft.fft2(torch.fft.ifftshift(z))).reshape(-1)


def _image64(X, N):
    """A Z^H F^H X."""
    z = torch.fft.fftshift(torch.fft.ifft2(torch.fft.ifftshift(X.view(2 * N, 2 * N)))) * (2 * N) ** 2
    return (z[N // 2:N // 2 + N, N // 2:N // 2 + N] * _apod64(N)).reshape(-1)


def _blocks(case, u, v, w):
    """Rows in blocks: cells and separable factors on a window of the grid that holds the kept taps."""
    N, Ng = case["N"], 2 * case["N"]
    wide = Ng if case["S"] == 0 else min(Ng, case["S"] + 40 + case["S"] % 2)
    step = max(256, min(8192, int(3e7) // max(Ng, wide * wide)))
    t = torch.arange(Ng, dtype=torch.float64, device="cuda") - Ng // 2
    j = torch.arange(wide, device="cuda")
    idx = (torch.arange(W, device="cuda")[:, None] - W // 2 + 1 + wide // 2 - j[None, :]) % Ng
    for r0 in range(0, len(u), step):
        uk, vk, wk = (_dev(a[r0:r0 + step]) for a in (u, v, w))
        c = torch.exp(1j * math.pi * (wk[:, None] * (t * (L / N)) ** 2))
        h = torch.fft.fft(torch.fft.ifftshift(c, dim=1)) / Ng
        ax = []
        for x in (vk, uk):
            xt = x * (2.0 * L)
            f = torch.floor(xt)
            d = (xt - f)[:, None] - (torch.arange(W, device="cuda") - W // 2 + 1)
            arg = 1.0 - (2.0 * d / W) ** 2
            wt = torch.where(arg >= 0, torch.special.i0(BETA * torch.sqrt(arg.clamp(min=0))), torch.zeros_like(arg))
            g = sum(wt[:, i, None] * h[:, idx[i]] for i in range(W))
            q = (f.long()[:, None] + Ng // 2 - wide // 2 + j) % Ng
            ax.append((q, g, (wt * wt).sum(1)))
        (qv, gv, tv), (qu, gu, tu) = ax
        yield dict(r0=r0, Ng=Ng, qv=qv, gv=gv, qu=qu, gu=gu, total=tv * tu)


def _full_rows(b, X):
    cols = b["qv"][:, :, None] * b["Ng"] + b["qu"][:, None, :]
    return torch.einsum("nb,nb->n", b["gv"], (X[cols] * b["gu"][:, None, :]).sum(2))


def _kept(b, E):
    """(row, column, value) of the block's kept taps: the largest energies that reach E of the row's total."""
    e = ((b["gv"].abs() ** 2)[:, :, None] * (b["gu"].abs() ** 2)[:, None, :]).flatten(1)
    srt = torch.sort(e, dim=1, descending=True)[0]
    k = torch.searchsorted(torch.cumsum(srt, 1), (E * b["total"])[:, None]).clamp(max=e.shape[1] - 1)
    keep = e >= torch.gather(srt, 1, k)
    at = keep.nonzero()
    r, p = at[:, 0], at[:, 1]
    n = b["qu"].shape[1]
    pv, pu = p // n, p % n
    return b["r0"] + r, b["qv"][r, pv] * b["Ng"] + b["qu"][r, pu], b["gv"][r, pv] * b["gu"][r, pu]


def _taps64(case, u, v, w):
    parts = [_kept(b, case["E"]) for b in _blocks(case, u, v, w)]
    return [torch.cat(z) for z in zip(*parts)]


def _cadd(n, at, val):
    out = torch.zeros(n, 2, dtype=torch.float64, device="cuda")
    return torch.view_as_complex(out.index_add_(0, at, torch.view_as_real(val)))


def _apply64(case, u, v, w, x, y):
    """(Phi x, Phi^H y) in the caller's order."""
    N, M = case["N"], len(u)
    X = _grid64(x, N)
    yo = torch.zeros(M, dtype=torch.complex128, device="cuda")
    Xo = torch.zeros(4 * N * N, dtype=torch.complex128, device="cuda")
    for b in _blocks(case, u, v, w):
        r, c, g = _kept(b, case["E"])
        yo += _cadd(M, r, g * X[c])
        Xo += _cadd(4 * N * N, c, g.conj() * y[r])
    return yo, _image64(Xo, N)


def _zorder(N, u, v, nearest):
    """Stable order of visibilities by the Z-order code of their cell."""
    code = np.zeros(len(u), dtype=np.int64)
    for x, odd in ((u, 0), (v, 1)):
        c = np.floor(np.asarray(x) * (2.0 * L) + (0.5 if nearest else 0.0)).astype(np.int64) + N
        c = c % (2 * N) if nearest else np.clip(c, 0, 2 * N - 1)
        for bit in range(12):
            code |= ((c >> bit) & 1) << (2 * bit + odd)
    return np.argsort(code, kind="stable")


def _exact_apply(case, seed):
    N, M = case["N"], case["M"]
    u, v, w = _uvw(N, M, _w_top(case), seed, 1, uniform=case["S"] == 0)
    y = _dev(_vis(M, seed, 5)).to(torch.complex128)
    x = _sky(N, seed, 2).to(torch.complex64).to(torch.complex128)
    if case["order"] == "caller":
        yo, xo = _apply64(case, u, v, w, x, y)
        return {"y": yo, "x": xo}
    p = _zorder(N, u, v, False)
    yo, xo = _apply64(case, u[p], v[p], w[p], x, y)
    return {"y": yo, "x": xo}


def _exact_batch(case, seed):
    N, ys, xs, at = case["N"], [], [], 0
    yin = _dev(_vis(sum(M for M, _ in _channels(case)), seed, 5)).to(torch.complex128)
    for c, (M, w_top) in enumerate(_channels(case)):
        u, v, w = _uvw(N, M, w_top, seed, 100 + c)
        p = _zorder(N, u, v, False)
        x = _sky(N, seed, 200 + c).to(torch.complex64).to(torch.complex128)
        yo, xo = _apply64(case, u[p], v[p], w[p], x, yin[at:at + M])
        ys.append(yo)
        xs.append(xo)
        at += M
    return {"y": torch.cat(ys), "x": torch.cat(xs)}


def _exact_build(case, seed):
    out = {k: None for k in ("rowptr", "col", "val", "perm", "tcolptr", "trow", "tval")}
    if case["taps"] != "c64":
        return out                                    # packed pairs: whole numbers
    u, v, w = _uvw_cells(case["N"], case["M"], _w_top(case), seed)
    p = _zorder(case["N"], u, v, False)
    r, c, g = _taps64(case, u[p], v[p], w[p])
    cells = 4 * case["N"] ** 2
    o = torch.argsort(r * cells + c)                  # rows in order, columns ascending
    r, c, g = r[o], c[o], g[o]
    out["val"] = g
    out["tval"] = g[torch.argsort(c * case["M"] + r)]  # cells in order, rows ascending
    return out


def _db8():
    """Daubechies low-pass filter with 8 vanishing moments (spectral factorisation, minimum phase)."""
    z = []
    for y in np.roots([math.comb(7 + k, k) for k in range(8)][::-1]):
        b = 1.0 - 2.0 * y
        d = np.sqrt(b * b - 1.0 + 0j)
        z.append(b + d if abs(b + d) < 1 else b - d)
    h = np.real(np.poly(np.concatenate([-np.ones(8), z])))
    return h * math.sqrt(2.0) / h.sum()


def _wavelet(N, levels):
    """The orthonormal analysis matrix of each level (side n x n)."""
    h = _db8()
    g = (-1.0) ** np.arange(16) * h[::-1]
    mats = []
    for lv in range(levels):
        n = N >> lv
        A = np.zeros((n, n))
        for k in range(n // 2):
            np.add.at(A[k], (2 * k + np.arange(16)) % n, h)
            np.add.at(A[n // 2 + k], (2 * k + np.arange(16)) % n, g)
        mats.append(_dev(A))
    return mats


def _exact_solve(case, seed):
    N, M = case["N"], case["M"]
    (u, v, w), y, eps = _solve_data(case, seed)
    y = y.to(torch.complex128)
    r, c, g = _taps64(case, u, v, w)
    mats = _wavelet(N, case["levels"])

    def phi(x):
        return _cadd(M, r, g * _grid64(x.to(torch.complex128), N)[c])

    def phit(z):
        return _image64(_cadd(4 * N * N, c, g.conj() * z[r]), N).real.view(N, N)

    def analysis(x):
        x = x.clone()
        for A in mats:
            n = A.shape[0]
            x[:n, :n] = A @ x[:n, :n] @ A.T
        return x

    def synthesis(x):
        x = x.clone()
        for A in reversed(mats):
            n = A.shape[0]
            x[:n, :n] = A.T @ x[:n, :n] @ A
        return x

    x = _dev(_start(case, seed)).double().view(N, N)
    x = x / x.norm()
    for _ in range(case["power"]):
        z = phit(phi(x))
        nu = float(z.norm())
        x = z / nu
    s2 = 1.0 / (1.05 * nu)
    x = torch.zeros(N, N, dtype=torch.float64, device="cuda")
    v1, v2 = torch.zeros_like(x), torch.zeros_like(y)
    for _ in range(case["iters"]):
        xn = (x - 0.49 * (synthesis(v1) + phit(v2))).clamp(min=0)
        xb = 2 * xn - x
        v1 = (v1 + analysis(xb)).clamp(-1, 1)
        p = v2 + s2 * phi(xb)
        res = p / s2 - y
        nr = float(res.norm())
        v2 = p - s2 * (y + res * min(1.0, eps / nr if nr > 0 else 1.0))
        x = xn
    return {"nu": nu, "x": x.reshape(-1)}


def _layers(params):
    out, at = [], 0
    for n, k in ((H, 3), (H, H), (H, H), (NOUT, H)):
        out += [params[at:at + n * k].view(n, k), params[at + n * k:at + n * k + n]]
        at += n * k + n
    return out


def _hidden(x, p):
    for i in range(3):
        x = torch.nn.functional.gelu(x @ p[2 * i].T + p[2 * i + 1])
    return x


def _exact_net(case, seed):
    params = _dev(_net(seed)).double()
    x = _dev(_features(case["n"], seed)).double()
    if case["kind"] == "infer":
        p = _layers(params)
        return {"out": (_hidden(x, p) @ p[6].T + p[7]).reshape(-1)}
    params.requires_grad_(True)
    p = _layers(params)
    loss = ((_hidden(x, p) @ p[6].T + p[7]).reshape(-1) - _targets(case["n"], seed).double()).square().mean()
    loss.backward()
    return {"grads": params.grad, "loss": float(loss.detach())}


def _exact_surrogate(case, seed):
    N, M, Ng = case["N"], case["M"], 2 * case["N"]
    u, v, w = _uvw(N, M, _w_top(case), seed, 1)
    over = _over_tol(case, seed) > TOL
    net, fb = np.flatnonzero(~over), np.flatnonzero(over)
    net = net[_zorder(N, u[net], v[net], True)]
    fb = fb[_zorder(N, u[fb], v[fb], False)]
    y = _dev(_vis(M, seed, 5)).to(torch.complex128)
    x = _sky(N, seed, 2).to(torch.complex64).to(torch.complex128)
    p = _layers(_dev(_net(seed)).double())
    X = _grid64(x, N)
    Xo = torch.zeros(Ng * Ng, dtype=torch.complex128, device="cuda")
    t = np.arange(-W // 2 + 1, W // 2 + 1)
    total = float((torch.special.i0(BETA * torch.sqrt(torch.clamp(1 - _dev((2.0 * t / W) ** 2), min=0))) ** 2).sum())
    s_out = total / BOX
    o = torch.arange(BOX, device="cuda") - BOX // 2
    yo = []
    for r0 in range(0, len(net), 8192):
        k = net[r0:r0 + 8192]
        ut, vt, wk = _dev(u[k] * 2.0 * L), _dev(v[k] * 2.0 * L), _dev(w[k])
        cu, cv = torch.floor(ut + 0.5), torch.floor(vt + 0.5)
        f = torch.stack([2 * wk / _w_top(case) - 1, 2 * (ut - cu), 2 * (vt - cv)], 1)
        taps = torch.view_as_complex((s_out * (_hidden(f, p) @ p[6].T + p[7])).view(len(k), BOX * BOX, 2))
        qv, qu = (cv.long()[:, None] + N + o) % Ng, (cu.long()[:, None] + N + o) % Ng
        cols = (qv[:, :, None] * Ng + qu[:, None, :]).flatten(1)
        yo.append((taps * X[cols]).sum(1))
        Xo += _cadd(Ng * Ng, cols.reshape(-1), (taps.conj() * y[r0:r0 + len(k), None]).reshape(-1))
    xo = _image64(Xo, N)
    if len(fb):
        yf, xf = _apply64(case, u[fb], v[fb], w[fb], x, y[len(net):])
        yo.append(yf)
        xo = xo + xf
    return {"y": torch.cat(yo), "x": xo}


def exact(case, seed):
    kind = case["kind"]
    with torch.no_grad() if kind != "train" else torch.enable_grad():
        return {"apply": _exact_apply, "batch": _exact_batch, "build": _exact_build, "solve": _exact_solve,
                "train": _exact_net, "infer": _exact_net, "surrogate": _exact_surrogate}[kind](case, seed)
