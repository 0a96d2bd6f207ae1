"""The work this library is used for, as measurable cases.

A case names one problem (patch, detectors, samples, noise model, precision,
columns) and one of these uses of it:

  apply     y = A x, the product every solver iteration repeats (forward
            gather, inverse-noise weight, map reduction)
  weight32  y = P x and z = N^-1 y in the FP32 form: the time-domain part of
            the inner solves of the precision form
  rhs       b = P^T N^-1 d: data to map, once per data set or realisation
  solve     whole preconditioned solves
  request   a served request: rhs, then an M_2l solve with the cached space
  register  what a new scan strategy costs: pointing, grid hint, noise, M_BD

Sizes are those of the benchmark's configurations (a 32 x 32 latency patch, a
256 x 256 patch with 2^27 samples, the serving strategies, template-filter and
detector-pair scans) and ragged ones beside them.
"""
import math

import numpy as np
import torch

from paper_1801_08937_amd import mapmaker as mm

F_SAMP = 20.0
CHUNK = 1 << 26  # elements of the largest temporary in exact()


def _case(name, kind, n_side, gx, gy, spd, L, lam, **kw):
    c = dict(name=name, kind=kind, n_side=n_side, gx=gx, gy=gy, spd=spd, L=L, lam=lam, R=1,
             prec="f64", stokes="IQU", weight="band", order=2, sub=256, ragged=False, grid=True,
             straight=False, filters="det", precond="mbd", min_hits=3)
    c.update(kw)
    return c


def listed():
    return [
        # the latency patch: 2 x 65,536 samples, everything in cache, direct band
        _case("patch32_apply", "apply", 32, 2, 1, 1 << 16, 1 << 14, 32, straight=True, grid=False,
              filters="one"),
        # 64 Monte Carlo realisations solved together on that patch
        _case("patch32_solve64", "solve", 32, 2, 1, 1 << 16, 1 << 14, 32, straight=True,
              grid=False, filters="one", R=64),
        # a small served request with a cached deflation space: 16 x 2^16 samples
        _case("serve64_request", "request", 64, 4, 4, 1 << 16, 1 << 16, 1024, precond="m2l"),
        # an ordinary strategy, one column: 32 x 2^18 samples
        _case("serve128_apply", "apply", 128, 8, 4, 1 << 18, 1 << 16, 2048),
        # the same in a session of four columns
        _case("serve128_apply_r4", "apply", 128, 8, 4, 1 << 18, 1 << 16, 2048, R=4),
        # the largest: 128 x 2^20 samples, half-bandwidth 4,096
        _case("patch256_apply", "apply", 256, 16, 8, 1 << 20, 1 << 16, 4096),
        # FP32 time-domain work of the precision form, 64 x 2^20 samples
        _case("patch256_f32", "weight32", 256, 8, 8, 1 << 20, 1 << 16, 4096, prec="f32"),
        # data to map on the 64-detector strategy
        _case("patch256_rhs", "rhs", 256, 8, 8, 1 << 20, 1 << 16, 4096),
        # polynomials per subscan and azimuth-binned ground templates
        _case("ground_apply", "apply", 256, 8, 4, 1 << 20, 1 << 20, 0, weight="ground"),
        # pair-difference stream (Q, U), offset and slope per subscan
        _case("pair_qu_apply", "apply", 256, 8, 4, 1 << 20, 1 << 20, 0, weight="poly", order=1,
              stokes="QU"),
        # a user's own scan: odd sizes, uneven intervals, no grid hint
        _case("ragged_apply", "apply", 101, 5, 3, 199999, 23000, 333, ragged=True, grid=False),
        # registering an ordinary strategy
        _case("serve128_register", "register", 128, 8, 4, 1 << 18, 1 << 16, 2048),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["apply"] * 6 + ["weight32", "weight32", "rhs", "rhs", "request", "solve",
                                       "register"])
    n_side = _log(rng, 24, 256)
    gx, gy = rng.choice([(2, 1), (3, 1), (4, 2), (4, 4), (5, 3), (8, 4), (8, 8), (16, 8)])
    weight, stokes, order, sub, R = "band", "IQU", 2, 256, 1
    if kind == "apply":
        weight = rng.choice(["band", "band", "band", "poly", "ground"])
        stokes = rng.choice(["IQU", "IQU", "I", "QU"]) if weight == "poly" else "IQU"
        order = rng.choice([0, 1, 2, 3])
        sub = rng.choice([64, 200, 256, 333, 512, 777])
        R = rng.choice([1, 1, 1, 2, 4, 8, 16, 64]) if weight == "band" else rng.choice([1, 1, 2])
    elif kind == "rhs":
        R = rng.choice([1, 1, 2, 8])
    elif kind == "solve":
        R = rng.choice([8, 16, 64])
    # total time-domain elements; enough hits for every pixel of the patch
    top = {"apply": 1 << 25, "weight32": 1 << 26, "rhs": 1 << 25, "request": 1 << 22,
           "solve": 1 << 23, "register": 1 << 24}[kind]
    n_det = gx * gy
    total = max(_log(rng, 1 << 17, top) // R, 24 * n_side * n_side)
    spd = max(total // n_det, 4096)
    if rng.random() < 0.5:
        spd = (spd + 63) // 64 * 64
    L = min(spd, rng.choice([1 << 12, 1 << 14, 1 << 16, 10000, 50001]))
    lam = min(_log(rng, 16, 8192), L // 4)
    straight = rng.random() < 0.3
    if kind == "solve":
        lam = min(lam, 256)
    c = _case("", kind, n_side, gx, gy, spd, L, lam, R=R, weight=weight, stokes=stokes,
              order=order, sub=sub, prec="f32" if kind == "weight32" else "f64",
              ragged=rng.random() < 0.4, grid=rng.random() < 0.7, straight=straight,
              filters=rng.choice(["det", "one"]), precond="m2l" if kind == "request" else "mbd")
    if weight != "band":
        c["L"], c["lam"], c["ragged"] = spd, 0, False
    del c["name"]
    return c


# ---------------------------------------------------------------- inputs

def _dev():
    return torch.device("cuda", 0)


def _scan(c):
    """pix int32[n], and the azimuth bin of each sample for ground templates."""
    n, gx, gy, spd = c["n_side"], c["gx"], c["gy"], c["spd"]
    nd, d = gx * gy, _dev()
    t = torch.arange(spd, device=d, dtype=torch.int64)
    pix = torch.empty(nd, spd, dtype=torch.int32, device=d)
    ground = c["weight"] == "ground"
    gb = torch.empty(nd, spd, dtype=torch.int32, device=d) if ground else None
    q, u = t // n, t % n
    m = q // n
    fwd = torch.where(q % 2 == 0, u, n - 1 - u)
    half = n / 2.0
    a = fwd.double() + 0.5 - half
    b = (q % n).double() + 0.5 - half
    th = (m % 3).double() * math.radians(60.0)
    if c["straight"]:
        th = torch.zeros_like(th)
    ct, st = torch.cos(th), torch.sin(th)
    x, y = half + a * ct - b * st, half + a * st + b * ct
    n_loc = n + 2 * (gx + gy)
    for k in range(nd):
        ox, oy = 2 * (k % gx) - (gx - 1), 2 * (k // gx) - (gy - 1)
        if c["straight"]:
            pix[k] = ((q + (n * k) // nd) % n * n + fwd).int()
        else:
            ix, iy = torch.floor(x + ox).long(), torch.floor(y + oy).long()
            ok = (ix >= 0) & (ix < n) & (iy >= 0) & (iy < n)
            pix[k] = torch.where(ok, iy * n + ix, torch.full_like(ix, -1)).int()
        if ground:
            az = torch.floor(a + ox * ct + oy * st + half + gx + gy).long().clamp(0, n_loc - 1)
            gb[k] = (m * n_loc + az).int()
    nb = int((spd - 1) // (n * n) + 1) * n_loc
    return pix.reshape(-1), (gb.reshape(-1) if ground else None), nb


def _gen(seed, stream):
    g = torch.Generator(device=_dev())
    g.manual_seed(1000003 * (int(seed) + 1) + stream)
    return g


def _band(L, lam, fknee):
    """Tapered inverse-noise coefficients of a 1/f spectrum, slope 1.7."""
    k = np.arange(L // 2 + 1, dtype=np.float64)
    g = np.zeros(L // 2 + 1)
    g[1:] = 1.0 / (1.0 + (fknee / (k[1:] * F_SAMP / L)) ** 1.7)
    ch = np.fft.irfft(g, n=2 * (L // 2))
    return ch[: lam + 1] * (1.0 - np.arange(lam + 1) / (lam + 1.0))


def _model(c, seed):
    """Intervals, filters and bands (or subscans and weights)."""
    r = np.random.default_rng([int(seed), 7])
    nd, spd, L = c["gx"] * c["gy"], c["spd"], c["L"]
    per = max(1, spd // L)
    cuts, fid = [0], []
    for k in range(nd):
        if c["ragged"] and per > 1:
            w = r.uniform(0.75, 1.25, per)
            e = np.floor(np.cumsum(w) / w.sum() * spd).astype(np.int64)
        else:
            e = np.arange(1, per + 1, dtype=np.int64) * L
        e[-1] = spd
        cuts += [int(v) + k * spd for v in e]
        fid += [k if c["filters"] == "det" else 0] * per
    m = dict(istart=np.asarray(cuts, dtype=np.int64), fid=np.asarray(fid, dtype=np.int32))
    nf = nd if c["filters"] == "det" else 1
    if c["weight"] == "band":
        m["band"] = np.stack([_band(L, c["lam"], f) for f in r.uniform(0.05, 1.0, nf)])
    else:
        m["w"] = r.uniform(0.5, 2.0, len(fid))
        m["sub"] = np.unique(np.concatenate(
            [np.arange(0, spd, c["sub"], dtype=np.int64) + k * spd for k in range(nd)]
            + [np.asarray([nd * spd])]))
    return m


def _psi(c, seed, n):
    return torch.rand(n, generator=_gen(seed, 1), device=_dev(), dtype=torch.float64) * math.pi


def _tod(c, seed, n):
    """[R][n] data: a sky signal's variance plus 1/f noise, per realisation."""
    g, R, nd, spd = _gen(seed, 2), c["R"], c["gx"] * c["gy"], c["spd"]
    out = torch.empty(R, n, dtype=torch.float64, device=_dev())
    N = 1 << (spd - 1).bit_length()
    f = torch.arange(N // 2 + 1, device=_dev(), dtype=torch.float64) * (F_SAMP / N)
    f[0] = f[1]
    shape = torch.sqrt(1.0 + (0.5 / f) ** 1.7)
    step = max(1, CHUNK // N)
    rows = out.view(R * nd, spd)
    for i in range(0, R * nd, step):
        w = torch.randn(min(step, R * nd - i), N, generator=g, device=_dev(), dtype=torch.float64)
        s = torch.fft.irfft(torch.fft.rfft(w) * shape, n=N)[:, :spd]
        rows[i:i + step] = s
        del w, s
    out += 100.0 * torch.randn(n, generator=g, device=_dev(), dtype=torch.float64)
    return out


def _map(c, seed, n):
    """A map vector of n = nc n_obs entries and R columns: I rms 100, Q, U 5."""
    v = torch.randn(n * c["R"], generator=_gen(seed, 3), device=_dev(), dtype=torch.float64)
    amp = {"IQU": [100.0, 5.0, 5.0], "I": [100.0], "QU": [5.0, 5.0]}[c["stokes"]]
    a = torch.tensor(amp, device=_dev(), dtype=torch.float64)
    return (v.view(-1, len(amp), c["R"]) * a[None, :, None]).reshape(-1).contiguous()


# ------------------------------------------------------------------- runs

def _noise(ctx, c, m, p, gb, nb):
    prec = mm.F32 if c["prec"] == "f32" else mm.F64
    if c["weight"] == "band":
        return ctx.noise(m["istart"], m["fid"], m["band"], c["lam"], mm.NOISE_AUTO, prec)
    return ctx.polyfilter(p, m["istart"], m["w"], m["sub"], c["order"],
                          ground_bin=gb, n_ground_bins=nb if gb is not None else 0)


def prepare(case, seed):
    c = case
    ctx = mm.Context(0)
    pix, gb, nb = _scan(c)
    psi = _psi(c, seed, pix.numel())
    m = _model(c, seed)
    prec = mm.F32 if c["prec"] == "f32" else mm.F64
    npix = c["n_side"] ** 2
    s = dict(c=c, ctx=ctx)
    if c["kind"] == "register":
        s.update(pix=pix, psi=psi, m=m, npix=npix, seed=seed)
        hits = torch.bincount(pix[pix >= 0].long(), minlength=npix)
        s["v"] = _map(c, seed, 3 * int((hits >= c["min_hits"]).sum()))
        return s
    p = ctx.pointing(pix, None if c["stokes"] == "I" else psi, npix, c["min_hits"], prec,
                     c["stokes"])
    if c["grid"]:
        p.set_grid(c["n_side"])
    nz = _noise(ctx, c, m, p, gb, nb)
    s.update(p=p, nz=nz)
    if c["kind"] in ("apply", "weight32"):
        s["x"] = _map(c, seed, p.n)
        if c["kind"] == "apply":
            s["y"] = torch.empty_like(s["x"])
        else:
            s["y"] = torch.empty(p.n_samp, dtype=torch.float32, device=_dev())
            s["z"] = torch.empty_like(s["y"])
        return s
    tod = _tod(c, seed, pix.numel()).reshape(-1)
    if c["kind"] == "rhs":
        s["tod"], s["b"] = tod, torch.empty(p.n * c["R"], dtype=torch.float64, device=_dev())
        return s
    M = ctx.mbd(p, nz)
    if c["kind"] == "solve":
        s.update(M=M, b=ctx.rhs(p, nz, tod, nrhs=c["R"]))
        return s
    b0 = ctx.rhs(p, nz, _tod(c, seed + 500009, pix.numel()).reshape(-1))
    s.update(mbd=M, tod=tod, M=ctx.defl_build(p, nz, M, b0, k=min(32, p.n // 8), eps_arn=1e-10,
                                              m_max=96, stop="residual"))
    return s


TOL = 1e-11  # tight, so that the maps compare beyond the stopping point


def run(state):
    s, c, ctx = state, state["c"], state["ctx"]
    kind = c["kind"]
    if kind == "apply":
        return ctx.apply_A(s["p"], s["nz"], s["x"], s["y"], nrhs=c["R"])
    if kind == "weight32":
        y = ctx.apply_P(s["p"], s["x"], s["y"])
        return y, ctx.noise_apply(s["nz"], y, s["z"])
    if kind == "rhs":
        return ctx.rhs(s["p"], s["nz"], s["tod"], s["b"], nrhs=c["R"])
    if kind == "solve":
        x, _ = ctx.solve(s["p"], s["nz"], s["M"], s["b"], tol=TOL, max_iter=500, nrhs=c["R"],
                         check_every=4, history=False)
        return x
    if kind == "request":
        b = ctx.rhs(s["p"], s["nz"], s["tod"])
        x, _ = ctx.solve(s["p"], s["nz"], s["M"], b, tol=TOL, max_iter=500, check_every=4,
                         history=False)
        return b, x
    p = ctx.pointing(s["pix"], s["psi"], s["npix"], c["min_hits"], mm.F64)
    if c["grid"]:
        p.set_grid(c["n_side"])
    m = s["m"]
    nz = ctx.noise(m["istart"], m["fid"], m["band"], c["lam"])
    M = ctx.mbd(p, nz)
    hits, obs = p.hits()
    j, perm, off = p.export()
    return hits, obs, j, perm, off, ctx.precond_apply(M, s["v"])


# ---------------------------------------------------- the least work of a pass

def work(case):
    c = case
    n, R, nd = c["gx"] * c["gy"] * c["spd"], c["R"], c["gx"] * c["gy"]
    te = 4 if c["prec"] == "f32" else 8
    nmap = {"IQU": 3, "I": 1, "QU": 2}[c["stokes"]] * c["n_side"] ** 2
    point = 4 + (0 if c["stokes"] == "I" else 8)  # pixel and angle of a sample
    if c["weight"] == "band":
        lam = c["lam"]
        # a real transform pair of blocks of about 8 lambda, or the band itself
        wf = min(4.0 * lam + 2, 7.0 * math.log2(max(8 * lam, 2)))
    else:
        wf = 8.0 * (c["order"] + 1) * (2 if c["weight"] == "ground" else 1)
    a_bytes = n * point + 16 * nmap * R
    a_flops = n * R * (10 + wf)
    if c["weight"] == "ground":
        a_bytes += 4 * n
    kind = c["kind"]
    if kind == "apply":
        return {"bytes": a_bytes, "flops": a_flops}
    if kind == "weight32":
        return {"bytes": n * point + 8 * nmap + 2 * te * n, "flops": n * (5 + wf)}
    if kind == "rhs":
        return {"bytes": n * (point + te * R) + 8 * nmap * R, "flops": n * R * (5 + wf)}
    if kind in ("solve", "request"):
        it = 20  # iterations that such a solve takes, about
        return {"bytes": it * (a_bytes + 80 * nmap * R), "flops": it * (a_flops + 30 * nmap * R)}
    return {"bytes": n * (12 + 8 + 4 + 4) + 4 * nd * 8 + 24 * nmap, "flops": 20 * n}


# ------------------------------------------------------------- exact values

def _weights(c, psi, n):
    one = torch.ones(n, dtype=torch.float64, device=_dev())
    if c["stokes"] == "I":
        return [one]
    cs = [torch.cos(2 * psi), torch.sin(2 * psi)]
    return cs if c["stokes"] == "QU" else [one] + cs


class _Exact:
    """A, b and M_BD of a case in torch, 64 bits."""

    def __init__(self, c, seed):
        self.c = c
        pix, gb, nb = _scan(c)
        self.n, npix = pix.numel(), c["n_side"] ** 2
        ok = pix >= 0
        self.hits = torch.bincount(pix[ok].long(), minlength=npix)
        seen = self.hits >= c["min_hits"]
        self.obs = torch.nonzero(seen).reshape(-1)
        comp = torch.full((npix,), -1, dtype=torch.int64, device=_dev())
        comp[self.obs] = torch.arange(self.obs.numel(), device=_dev())
        self.j = torch.where(ok, comp[pix.clamp(min=0).long()], torch.full((1,), -1, device=_dev()))
        self.on = self.j >= 0
        self.jc = self.j.clamp(min=0)
        self.n_obs = self.obs.numel()
        self.w = _weights(c, _psi(c, seed, self.n), self.n)
        self.nc = len(self.w)
        self.m = _model(c, seed)
        self.gb, self.nb = gb, nb

    def P(self, x):  # [n_obs, nc, R] -> [n, R]
        y = 0
        for a in range(self.nc):
            y = y + self.w[a][:, None] * x[:, a, :][self.jc]
        return torch.where(self.on[:, None], y, torch.zeros((), device=_dev(), dtype=y.dtype))

    def PT(self, z):
        out = torch.zeros(self.n_obs, self.nc, z.shape[1], dtype=torch.float64, device=_dev())
        z = torch.where(self.on[:, None], z, torch.zeros((), device=_dev(), dtype=z.dtype))
        for a in range(self.nc):
            t = torch.zeros(self.n_obs, z.shape[1], dtype=torch.float64, device=_dev())
            out[:, a, :] = t.index_add_(0, self.jc, self.w[a][:, None] * z)
        return out

    def rows(self, start, count):
        s = torch.from_numpy(start[:-1]).to(_dev())
        ln = torch.from_numpy(np.diff(start)).to(_dev())
        k = torch.arange(count, device=_dev())
        return s[:, None] + k[None, :], k[None, :] < ln[:, None]

    def N(self, y):
        if self.c["weight"] != "band":
            return torch.stack([self.F(y[:, r]) for r in range(y.shape[1])], 1)
        ist, lam, R = self.m["istart"], self.c["lam"], y.shape[1]
        Lm = int(np.diff(ist).max())
        N = 1 << (Lm + lam - 1).bit_length()
        if N * 3 // 4 >= Lm + lam:
            N = N * 3 // 4
        h = torch.zeros(self.m["band"].shape[0], N, dtype=torch.float64, device=_dev())
        bd = torch.from_numpy(self.m["band"]).to(_dev())
        h[:, : lam + 1] = bd
        if lam:
            h[:, N - lam:] = bd[:, 1:].flip(1)
        H = torch.fft.rfft(h).real
        fid = torch.from_numpy(self.m["fid"].astype(np.int64)).to(_dev())
        z = torch.empty_like(y)
        step = max(1, CHUNK // (2 * N * R))
        for i in range(0, len(ist) - 1, step):
            idx, ok = self.rows(ist[i:i + step + 1], Lm)
            v = torch.where(ok[..., None], y[idx.clamp(max=self.n - 1)],
                            torch.zeros((), device=_dev(), dtype=y.dtype))
            v = torch.fft.rfft(v, n=N, dim=1) * H[fid[i:i + step]][..., None]
            v = torch.fft.irfft(v, n=N, dim=1)[:, :Lm]
            z[idx[ok]] = v[ok]
        return z

    def sample_w(self):
        w = torch.from_numpy(self.m["w"]).to(_dev())
        ln = torch.from_numpy(np.diff(self.m["istart"])).to(_dev())
        return torch.where(self.on, torch.repeat_interleave(w, ln),
                           torch.zeros((), device=_dev(), dtype=torch.float64))

    def fit(self, y, w):
        """y minus each subscan's weighted polynomial fit, 0 where w is."""
        sub, NP = self.m["sub"], self.c["order"] + 1
        Lm = int(np.diff(sub).max())
        ln = torch.from_numpy(np.diff(sub)).to(_dev())
        out = torch.zeros_like(y)
        step = max(1, CHUNK // (Lm * (NP + 2)))
        for i in range(0, len(sub) - 1, step):
            idx, ok = self.rows(sub[i:i + step + 1], Lm)
            idc = idx.clamp(max=self.n - 1)
            k = torch.arange(Lm, device=_dev(), dtype=torch.float64)
            u = (2 * k[None, :] + 1) / ln[i:i + step, None] - 1
            B = [torch.ones_like(u), u]
            for d in range(2, NP):
                B.append(((2 * d - 1) * u * B[-1] - (d - 1) * B[-2]) / d)
            B = B[:NP]
            zero = torch.zeros((), device=_dev(), dtype=torch.float64)
            wv, yv = torch.where(ok, w[idc], zero), torch.where(ok, y[idc], zero)
            G = torch.stack([torch.stack([(wv * p * q).sum(1) for q in B], 1) for p in B], 1)
            g = torch.stack([(wv * p * yv).sum(1) for p in B], 1)
            live = (wv > 0).sum(1) > NP
            G = torch.where(live[:, None, None], G, torch.eye(NP, device=_dev(), dtype=G.dtype))
            a = torch.linalg.solve(G, g[..., None])[..., 0]
            res = yv - sum(a[:, d:d + 1] * B[d] for d in range(NP))
            res = torch.where(live[:, None] & (wv > 0), res, zero)
            out[idx[ok]] = res[ok]
        return out

    def F(self, y):
        w = self.sample_w()
        v = self.fit(y, w)
        if self.gb is not None:
            b, inb = self.gb.clamp(min=0).long(), self.gb >= 0
            wb = torch.where(inb, w, torch.zeros_like(w))
            tot = torch.zeros(self.nb, dtype=torch.float64, device=_dev()).index_add_(0, b, wb)
            sm = torch.zeros_like(tot).index_add_(0, b, wb * v)
            mean = torch.where(tot > 0, sm / tot, torch.zeros_like(tot))
            v = torch.where(inb & (w > 0), v - mean[b], v)
            v = self.fit(v, w)
        return w * v

    def A(self, x):
        return self.PT(self.N(self.P(x)))

    def rhs(self, tod):
        z = torch.zeros((), device=_dev(), dtype=torch.float64)
        return self.PT(self.N(torch.where(self.on[:, None], tod.t().contiguous(), z)))

    def mbd(self):
        c0 = torch.from_numpy(self.m["band"][self.m["fid"], 0]).to(_dev())
        ln = torch.from_numpy(np.diff(self.m["istart"])).to(_dev())
        w = torch.where(self.on, torch.repeat_interleave(c0, ln), torch.zeros_like(self.w[0]))
        B = torch.zeros(self.n_obs, self.nc, self.nc, dtype=torch.float64, device=_dev())
        for a in range(self.nc):
            for b in range(a, self.nc):
                t = torch.zeros(self.n_obs, dtype=torch.float64, device=_dev())
                t.index_add_(0, self.jc, w * self.w[a] * self.w[b])
                B[:, a, b] = t
                B[:, b, a] = t
        return torch.linalg.inv(B)

    def solve(self, b):
        """Conjugate gradients with M_BD to a 1e-14 residual."""
        Mi = self.mbd()
        pre = lambda r: (Mi[..., None] * r[:, None, :, :]).sum(2)  # noqa: E731
        dot = lambda u, v: (u * v).sum((0, 1))  # noqa: E731
        x, r = torch.zeros_like(b), b.clone()
        z = pre(r)
        p, rho, b2 = z.clone(), dot(r, z), dot(b, b)
        for _ in range(300):
            q = self.A(p)
            al = rho / dot(p, q)
            x, r = x + al * p, r - al * q
            if bool((dot(r, r) <= 1e-28 * b2).all()):
                break
            z = pre(r)
            new = dot(r, z)
            p, rho = z + (new / rho) * p, new
        return x


def exact(case, seed):
    c = case
    E = _Exact(c, seed)
    kind, R = c["kind"], c["R"]
    if kind == "register":
        Mi = E.mbd()
        v = _map(c, seed, 3 * E.n_obs).view(E.n_obs, 3)
        return None, None, None, None, None, (Mi * v[:, None, :]).sum(2).reshape(-1)
    if kind in ("apply", "weight32"):
        x = _map(c, seed, E.nc * E.n_obs).view(E.n_obs, E.nc, R)
        if kind == "apply":
            return E.A(x).reshape(-1)
        y = E.P(x)
        return y.reshape(-1), E.N(y).reshape(-1)
    b = E.rhs(_tod(c, seed, E.n))
    if kind == "rhs":
        return b.reshape(-1)
    if E.n * R > (1 << 24):
        return None if kind == "solve" else (b.reshape(-1), None)
    x = E.solve(b).reshape(-1)
    return x if kind == "solve" else (b.reshape(-1), x)
