"""Performance cases of the radiative-transfer library: the work its users have it do.

Every case goes through the public entry points of ``paper_2102_01734_amd``
(``Grid`` / ``SphereGrid``) as a program that owns a grid handle calls them:
formal solutions (one or several wavelengths, with or without Lambda*, over all
directions or one GPU's share of them), ALI steps replayed as HIP graphs, whole
solves, the nearest-neighbour Lambda* stencil and the learned correction's
network.  ``exact`` evaluates the same operators in 64 bits with plain torch
and numpy, from the definitions (quadrature, characteristics, weights), without
the library.

A case is a dict of plain values; ``kind`` names the path:

* ``box_fs``      formal solution on the periodic box (``shards`` > 1: the
                  directions of one of that many GPUs)
* ``box_step``    one ALI step over a wavelength batch, graph replay
* ``box_solve``   a whole ``solve`` from J = B
* ``box_stencil`` nearest-neighbour Lambda*
* ``sphere_fs``   formal solution on the spherical grid
* ``net``         network inference of the learned correction

Single-precision programs hand J and S on in the precision of their fields, so
the float64 state of a single-precision ALI step or solve is returned in it.
"""
import math

import numpy as np
import torch

import paper_2102_01734_amd as rt

# Algorithmic operations of one characteristic point: optical step 3, exp 1,
# moments 5, reciprocal 4, the three weights 15, intensity update 8, J 2.
FLOPS_PER_POINT = 38
MAX_EXACT_POINTS = 3e9


def listed():
    box = dict(kind="box_fs", shards=1, lam=1)
    return [
        # smallest call: the boxes of a unit test or of a code being ported; launches and latency
        dict(box, name="fs_box_9_f64", nx=9, ny=9, nz=8, n_mu=4, n_phi=8, prec="f64", lstar="linear"),
        # first formal solution (J and Lambda*) of the 33^3 double-precision slab
        dict(box, name="fs_box_33_f64", nx=33, ny=33, nz=33, n_mu=8, n_phi=16, prec="f64", lstar="linear"),
        # ragged box, three wavelengths, the directions of one of four GPUs, parabolic Lambda*
        dict(box, name="fs_box_ragged_f32", nx=70, ny=53, nz=61, n_mu=16, n_phi=24, prec="f32", lam=3, shards=4,
             lstar="parabolic"),
        # the single-wavelength 129^3 x 2048-direction formal solution of every plain ALI step
        dict(box, name="fs_box_129_f32", nx=129, ny=129, nz=129, n_mu=32, n_phi=64, prec="f32", lstar="none"),
        # the largest box: layers wider than one LDS tile
        dict(box, name="fs_box_257_f32", nx=257, ny=257, nz=257, n_mu=32, n_phi=16, prec="f32", lstar="none"),
        # a wavelength batch of uneven optical depth, one ALI step per pass (NLTE continuum batch)
        dict(name="step_batch_129_f32", kind="box_step", nx=129, ny=129, nz=129, n_mu=16, n_phi=16, prec="f32",
             lam=16),
        # the double-precision slab solved to 1e-8 with Ng acceleration
        dict(name="solve_33_f64", kind="box_solve", nx=33, ny=33, nz=33, n_mu=8, n_phi=16, prec="f64",
             nonlocal_lstar=False, method="ali", tol=1e-8),
        # defect-corrected single-precision solve with the nearest-neighbour Lambda*
        dict(name="solve_65_nonlocal_f32", kind="box_solve", nx=65, ny=65, nz=65, n_mu=16, n_phi=32, prec="f32",
             nonlocal_lstar=True, method="ali", tol=1e-6),
        # building the nearest-neighbour Lambda* of a new opacity
        dict(name="stencil_97_f32", kind="box_stencil", nx=97, ny=97, nz=65, n_mu=16, n_phi=16, prec="f32", lam=1,
             lstar="linear"),
        # irradiated shell, 16 wavelengths per characteristic
        dict(name="fs_sphere_batch_f32", kind="sphere_fs", nr=49, nt=33, np=65, n_mu=8, n_phi=16, prec="f32", lam=16,
             lstar="none"),
        # small double-precision shell, one wavelength, J and Lambda*
        dict(name="fs_sphere_small_f64", kind="sphere_fs", nr=25, nt=17, np=34, n_mu=4, n_phi=8, prec="f64", lam=1,
             lstar="linear"),
        # one proposal of the learned correction on the benchmark's box
        dict(name="net_129", kind="net", nx=129, ny=129, nz=129, channels="16,32,32"),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case of the listed ranges, bounded by the listed cases' work."""
    kind = rng.choice(["box_fs", "box_fs", "box_fs", "box_step", "box_solve", "box_stencil", "sphere_fs",
                       "sphere_fs", "net"])
    prec = rng.choice(["f32", "f32", "f64"])
    lstar = rng.choice(["none", "none", "linear", "parabolic"])
    while True:
        box = dict(kind=kind, nx=_log_int(rng, 6, 200), ny=_log_int(rng, 6, 200), nz=_log_int(rng, 5, 150),
                   n_mu=2 * rng.randint(2, 12), n_phi=_log_int(rng, 4, 48), prec=prec)
        if kind == "box_fs":
            c = dict(box, lam=_log_int(rng, 1, 12), lstar=lstar, shards=rng.choice([1, 1, 1, 2, 4, 8]))
            most = 2.0e10
        elif kind == "box_step":
            c = dict(box, lam=_log_int(rng, 1, 16))
            most = 1.0e10
        elif kind == "box_solve":
            c = dict(box, nonlocal_lstar=rng.random() < 0.4, method="ali", tol=1e-8 if prec == "f64" else 1e-6)
            most = 3.0e8
        elif kind == "box_stencil":
            c = dict(box, lam=_log_int(rng, 1, 4), lstar=rng.choice(["linear", "parabolic"]))
            most = 3.0e9
        elif kind == "sphere_fs":
            c = dict(kind=kind, nr=_log_int(rng, 6, 60), nt=_log_int(rng, 5, 40), np=_log_int(rng, 6, 70),
                     n_mu=2 * rng.randint(1, 4), n_phi=_log_int(rng, 4, 16), prec=prec, lam=_log_int(rng, 1, 16),
                     lstar=lstar)
            most = 1.0e9
        else:
            c = dict(kind=kind, nx=_log_int(rng, 17, 160), ny=_log_int(rng, 17, 160), nz=_log_int(rng, 17, 160),
                     channels=rng.choice(["16,32,32", "16,32,64,64"]))
            if c["nx"] * c["ny"] * c["nz"] <= 129 ** 3:
                return c
            continue
        voxels = c["nx"] * c["ny"] * c["nz"] if "nx" in c else c["nr"] * c["nt"] * c["np"]
        if 2e5 < _points(c) <= most and voxels * c.get("lam", 1) <= 4e7:
            return c


# ---------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------
def _gen(seed, salt):
    g = torch.Generator(device="cuda")
    g.manual_seed(1000003 * int(seed) + salt)
    return g


def _uniform(gen, shape, lo, hi):
    return lo + (hi - lo) * torch.rand(shape, generator=gen, device="cuda", dtype=torch.float64)


def _stratified(n, tau_min, tau_max):
    """Opacity per layer whose optical depth is log-uniform over [tau_min, tau_max], top layer first."""
    r = (tau_max / tau_min) ** (1.0 / (n - 1))
    tau = tau_min * r ** torch.arange(n, dtype=torch.float64, device="cuda")
    return tau * (math.sqrt(r) - 1.0 / math.sqrt(r))


def _correlated(shape, ell, gen):
    """Zero-mean, unit-variance field of correlation exp(-d^2 / 2 ell^2), periodic in x and y."""
    nz, ny, nx = shape
    f = torch.fft.rfftn(torch.randn((2 * nz, ny, nx), generator=gen, device="cuda", dtype=torch.float64))
    for axis, n in enumerate((2 * nz, ny, nx)):
        d = torch.arange(n, dtype=torch.float64, device="cuda")
        k = torch.exp(-0.5 * (torch.minimum(d, n - d) / (ell / math.sqrt(2.0))) ** 2)
        k = torch.fft.rfft(k) if axis == 2 else torch.fft.fft(k)
        f = f * k.reshape([-1 if a == axis else 1 for a in range(3)])
    g = torch.fft.irfftn(f, s=(2 * nz, ny, nx))[:nz]
    return (g - g.mean()) / g.std()


def _dtype(case):
    return torch.float32 if case["prec"] == "f32" else torch.float64


def _box_fields(case, seed):
    """chi, eps, B, S, I_bc of a log-normal stratified box in the grid precision; a batch has uneven optical depths."""
    n, shape = case.get("lam", 1), (case["nz"], case["ny"], case["nx"])
    gen = _gen(seed, 1)
    chi = _stratified(shape[0], 1e-4, 1e4)[:, None, None] * 10.0 ** _correlated(shape, 8.0, gen)
    scale = 10.0 ** _uniform(gen, (n, 1, 1, 1), -3.0, 3.0) if n > 1 else torch.ones((1, 1, 1, 1), device="cuda")
    eps = 10.0 ** _uniform(gen, (n,) + shape, -4.0, 0.0)
    S = _uniform(gen, (n,) + shape, 0.2, 1.0)
    bc = torch.tensor([[0.0, 1.0]], device="cuda").repeat(n, 1)
    t = _dtype(case)
    return [x.to(t).contiguous() for x in (chi[None] * scale, eps, torch.ones_like(S), S, bc)]


def _sphere_fields(case, seed):
    """chi, S, I_bc of an irradiated shell: radial optical depth log-uniform over 1e-6..1e6, small scatter."""
    n, shape = case["lam"], (case["np"], case["nt"], case["nr"])
    gen = _gen(seed, 2)
    chi = torch.flip(_stratified(case["nr"], 1e-6, 1e6), [0]) * case["nr"]
    chi = chi * 10.0 ** (0.2 * torch.randn(shape, generator=gen, device="cuda", dtype=torch.float64))
    scale = 10.0 ** _uniform(gen, (n, 1, 1, 1), -2.0, 2.0)
    S = _uniform(gen, (n,) + shape, 0.2, 1.0)
    bc = torch.tensor([[0.0, 1.0, 1.0]], device="cuda").repeat(n, 1)
    t = _dtype(case)
    return [x.to(t).contiguous() for x in (chi[None] * scale, S, bc)]


def _net_channels(case):
    return [int(c) for c in case["channels"].split(",")]


def _net_layers(case, seed):
    """(taps, c_in, c_out, weights, biases) of every convolution in blob order."""
    C = _net_channels(case)
    L = len(C)
    pairs = [(27, 3, C[0]), (27, C[0], C[0])]
    for k in range(1, L):
        pairs += [(27, C[k - 1], C[k]), (27, C[k], C[k])]
    for k in range(L - 1, 0, -1):
        pairs += [(27, C[k], C[k - 1]), (27, C[k - 1], C[k - 1])]
    pairs.append((1, C[0], 1))
    rng = np.random.default_rng(7919 * int(seed) + 3)
    out = []
    for taps, ci, co in pairs:
        w = (rng.standard_normal((taps, co, ci)) * math.sqrt(1.0 / (taps * ci))).astype(np.float32)
        out.append((taps, ci, co, w, (0.05 * rng.standard_normal(co)).astype(np.float32)))
    return out


def _net_features(case, seed):
    gen = _gen(seed, 4)
    shape = (case["nz"], case["ny"], case["nx"])
    f = [_uniform(gen, shape, -1.0, 1.0), _uniform(gen, shape, -1.0, 1.0), _uniform(gen, shape, -1.0, 1.0)]
    return torch.stack(f, dim=-1).to(torch.float32).contiguous()


# ---------------------------------------------------------------------------
# what a program holds before the call, and the call
# ---------------------------------------------------------------------------
def prepare(case, seed):
    kind = case["kind"]
    if kind == "sphere_fs":
        lstar = "parabolic" if case["lstar"] == "parabolic" else "linear"
        g = rt.SphereGrid(case["nr"], case["nt"], case["np"], 1.0, 2.0, case["n_mu"], case["n_phi"], case["prec"],
                          case["lam"], lstar=lstar, source_distance=5.0)
        return dict(case=case, grid=g, fields=_sphere_fields(case, seed))
    if kind == "net":
        g = rt.Grid(case["nx"], case["ny"], case["nz"], 2, 4, "f32", 1)
        layers = _net_layers(case, seed)
        C = _net_channels(case)
        blob = b"RTUN" + np.asarray([1, len(C)] + C, dtype="<u4").tobytes()
        blob += b"".join(w.astype("<f4").tobytes() + b.astype("<f4").tobytes() for _, _, _, w, b in layers)
        g.set_preconditioner(blob)
        return dict(case=case, grid=g, features=_net_features(case, seed))
    g = rt.Grid(case["nx"], case["ny"], case["nz"], case["n_mu"], case["n_phi"], case["prec"], case.get("lam", 1),
                lstar="parabolic" if case.get("lstar") == "parabolic" else "linear",
                nonlocal_lstar=bool(case.get("nonlocal_lstar")))
    chi, eps, B, S, bc = _box_fields(case, seed)
    state = dict(case=case, grid=g)
    if kind == "box_fs":
        state.update(fields=[chi, S, bc])
        if case["shards"] > 1:
            state.update(dirs=g.shard_directions(case["shards"], 0))
    elif kind == "box_step":
        # a step of a solve whose iteration goes on: graph replays on the program's own stream
        state.update(ali=g.new_state(chi, eps, B, bc), stream=torch.cuda.Stream(),
                     opts=g.opts(tol=1e-30, max_iter=1, ng_every=4, ng_start=4, use_graph=True))
    elif kind == "box_solve":
        state.update(fields=[chi, eps, B, bc], opts=g.opts(tol=case["tol"], max_iter=60, method=case["method"]))
    else:
        state.update(chi=chi)
    return state


def run(state):
    case, g = state["case"], state["grid"]
    kind = case["kind"]
    if kind in ("box_fs", "sphere_fs"):
        chi, S, bc = state["fields"]
        want = case["lstar"] != "none"
        if "dirs" in state:
            J, L = g.formal_solution_dirs(chi, S, state["dirs"], bc, want_lstar=want)
        else:
            J, L = g.formal_solution(chi, S, bc, want_lstar=want)
        return dict(J=J, lstar=L) if want else dict(J=J)
    if kind == "box_step":
        st, s = state["ali"], state["stream"]
        s.wait_stream(torch.cuda.current_stream())
        with torch.cuda.stream(s):
            g.ali_step(st, state["opts"], stream=s)
        torch.cuda.current_stream().wait_stream(s)
        t = g.state_tensors(st)
        return dict(J=t["J"].to(_dtype(case)), S=t["S"].to(_dtype(case)), lstar=t["lstar"])
    if kind == "box_solve":
        chi, eps, B, bc = state["fields"]
        st = g.new_state(chi, eps, B, bc)
        g.solve(st, state["opts"])
        t = g.state_tensors(st)
        return dict(J=t["J"].to(_dtype(case)), S=t["S"].to(_dtype(case)))
    if kind == "box_stencil":
        return g.lstar_stencil(state["chi"])
    return g.precond_forward(state["features"])


# ---------------------------------------------------------------------------
# the work of one pass
# ---------------------------------------------------------------------------
def _direction(i, j, n_mu, n_phi):
    mu, phi = -1.0 + (2.0 * i + 1.0) / n_mu, 2.0 * math.pi * (j + 0.5) / n_phi
    st = math.sqrt(1.0 - mu * mu)
    return st * math.cos(phi), st * math.sin(phi), mu


def _points(case):
    """Characteristic points of one formal solution (an estimate on the sphere: about 4.6 visits per voxel)."""
    lam = case.get("lam", 1)
    if case["kind"] == "sphere_fs":
        return 4.6 * lam * case["nr"] * case["nt"] * case["np"] * case["n_mu"] * case["n_phi"]
    total = 0.0
    for i in range(case["n_mu"]):
        for j in range(case["n_phi"]):
            nx, ny, nz = _direction(i, j, case["n_mu"], case["n_phi"])
            t = case["nz"] / abs(nz)
            total += case["nz"] + math.floor(t * abs(nx) + 0.5) + math.floor(t * abs(ny) + 0.5)
    return total * case["nx"] * case["ny"] * lam / case.get("shards", 1)


def work(case):
    kind = case["kind"]
    if kind == "net":
        C, layers = _net_channels(case), _net_layers(case, 0)
        n = [case["nx"] * case["ny"] * case["nz"]]
        d = (case["nx"], case["ny"], case["nz"])
        for _ in C[1:]:
            d = tuple((x + 1) // 2 for x in d)
            n.append(d[0] * d[1] * d[2])
        level = [0, 0]
        for k in range(1, len(C)):
            level += [k, k]
        for k in range(len(C) - 1, 0, -1):
            level += [k - 1, k - 1]
        level.append(0)
        flops = sum(2.0 * t * ci * co * n[l] for (t, ci, co, _, _), l in zip(layers, level))
        return dict(bytes=n[0] * 16.0, flops=flops)
    e = 4 if case["prec"] == "f32" else 8
    lam = case.get("lam", 1)
    vox = lam * (case["nx"] * case["ny"] * case["nz"] if "nx" in case else case["nr"] * case["nt"] * case["np"])
    pts = _points(case)
    if kind in ("box_fs", "sphere_fs"):
        out = 1 if case["lstar"] == "none" else 2
        return dict(bytes=float(vox * e * (2 + out)), flops=FLOPS_PER_POINT * pts)
    if kind == "box_step":
        return dict(bytes=float(vox * (4 * e + 4 * 8)), flops=FLOPS_PER_POINT * pts)
    if kind == "box_solve":  # about 20 formal solutions
        return dict(bytes=float(vox * (3 * e + 2 * e)), flops=20.0 * FLOPS_PER_POINT * pts)
    return dict(bytes=float(vox * e * 28), flops=FLOPS_PER_POINT * pts)


# ---------------------------------------------------------------------------
# the same in 64 bits, from the definitions
# ---------------------------------------------------------------------------
def _moments(D):
    """exp(-D), e0 = 1 - exp(-D), e1 = D - e0, e2 = D^2 - 2 e1 without cancellation for small D."""
    ex = torch.exp(-D)
    e0 = -torch.expm1(-D)
    p = torch.zeros_like(D)
    for k in range(16, 2, -1):
        p = 1.0 / math.factorial(k) - D * p
    small = D < 0.25
    e2s = 2.0 * D ** 3 * p
    e1 = torch.where(small, 0.5 * (D * D - e2s), D - e0)
    return ex, e0, e1, torch.where(small, e2s, D * D - 2.0 * e1)


def _weights(D, Dn, last):
    """Weights of the previous, current and next source (parabolic, or linear where that is called for)."""
    D = torch.clamp(D, min=1e-100)
    ex, e0, e1, e2 = _moments(D)
    lin = last | (Dn < 0.5 * D) | (Dn * e0 <= D * e1 - e2)
    Dq = torch.where(lin, torch.ones_like(Dn), Dn)
    bl = e1 / D
    b = torch.where(lin, bl, ((D + Dq) * e1 - e2) / (D * Dq))
    g = torch.where(lin, torch.zeros_like(b), (e2 - D * e1) / (Dq * (D + Dq)))
    return ex, e0 - b - g, b, g, bl


def _sweep(M, at, n_pts, I0, parabolic, deposit):
    """Integrates a set of rays over up to M points; at(m) -> chi, S, s, and
    deposit(m, active, I, lambda_star_term) receives every point."""
    chi, S, s = at(0)
    t = chi * s
    ex, e0, _, _ = _moments(torch.clamp(0.5 * t, min=1e-100))
    I = I0 * ex + S * e0
    deposit(0, n_pts > 0, I, e0)
    Sp, tp, gp = S, t, torch.zeros_like(I)
    if M < 2:
        return
    chi, S, s = at(1)
    t = chi * s
    for m in range(1, M):
        last = n_pts <= m + 1
        Sn, tn = S, t
        if m + 1 < M:
            chi, Sn, s = at(m + 1)
            tn = chi * s
        ex, a, b, g, bl = _weights(0.5 * (tp + t), 0.5 * (t + tn), last.expand_as(t))
        I = I * ex + a * Sp + b * S + g * Sn
        deposit(m, n_pts > m, I, b + gp * ex if parabolic else bl)
        Sp, tp, S, t, gp = S, t, Sn, tn, g


def _box_template(nz, n):
    """Voxel offsets, layer and path length of the ray through the centre of the inflow face of column (0, 0)."""
    ax, ay, az = (abs(c) for c in n)
    T = nz / az
    kz = np.arange(1, nz + 1) / az
    tx = (np.arange(int(T * ax + 2)) + 0.5) / ax if ax > 0 else np.empty(0)
    ty = (np.arange(int(T * ay + 2)) + 0.5) / ay if ay > 0 else np.empty(0)
    t = np.concatenate([kz, tx[tx < kz[-1]], ty[ty < kz[-1]]])
    t.sort()
    ends, prev = [], 0.0
    for v in t.tolist():
        if v - prev > 1e-12 * (prev + 1.0):
            ends.append(v)
            prev = v
    e = np.asarray(ends)
    b = np.concatenate([[0.0], e[:-1]])
    mid = 0.5 * (b + e)
    i = np.searchsorted(tx, mid).astype(np.int64)
    j = np.searchsorted(ty, mid).astype(np.int64)
    k = np.minimum(np.searchsorted(kz, mid), nz - 1).astype(np.int64)
    di, dj = i if n[0] >= 0 else -i, j if n[1] >= 0 else -j
    return di, dj, k if n[2] < 0 else nz - 1 - k, e - b


def _lightest_shard(lengths, shards):
    """The directions of shard 0: dealt longest first to the shard with the fewest visits."""
    load, mine = [0] * shards, []
    for d in sorted(range(len(lengths)), key=lambda d: -lengths[d]):
        k = min(range(shards), key=lambda q: (load[q], q))
        load[k] += lengths[d]
        if k == 0:
            mine.append(d)
    return sorted(mine)


def _box_batches(case):
    """(di, dj, layer, s, visits, w |mu|, mu) of the directions, in groups of similar length."""
    n_mu, n_phi = case["n_mu"], case["n_phi"]
    ns = [_direction(i, j, n_mu, n_phi) for i in range(n_mu) for j in range(n_phi)]
    tpl = [_box_template(case["nz"], n) for n in ns]
    mine = list(range(len(ns)))
    if case.get("shards", 1) > 1:
        mine = _lightest_shard([len(t[3]) for t in tpl], case["shards"])
    mine.sort(key=lambda d: len(tpl[d][3]))
    per = max(1, int(1.5e6 / (case["nx"] * case["ny"] * case.get("lam", 1))))
    for k in range(0, len(mine), per):
        group = mine[k:k + per]
        M = max(len(tpl[d][3]) for d in group)

        def padded(c, kind):
            a = np.zeros((len(group), M), dtype=kind)
            for r, d in enumerate(group):
                v = tpl[d][c]
                a[r, :len(v)] = v
                a[r, len(v):] = v[-1]
            return torch.from_numpy(a).cuda()

        yield (padded(0, np.int64), padded(1, np.int64), padded(2, np.int64), padded(3, np.float64),
               torch.tensor([len(tpl[d][3]) for d in group], device="cuda"),
               torch.tensor([abs(ns[d][2]) / len(ns) for d in group], dtype=torch.float64, device="cuda"),
               torch.tensor([ns[d][2] for d in group], dtype=torch.float64, device="cuda"))


def _exact_box_fs(case, seed):
    chi, _, _, S, bc = (x.double() for x in _box_fields(case, seed))
    return _box_operator(case, chi, S, bc)


def _box_operator(case, chi, S, bc):
    nx, ny, nz, lam = case["nx"], case["ny"], case["nz"], case.get("lam", 1)
    chi, S = chi.reshape(lam, -1), S.reshape(lam, -1)
    J, L = torch.zeros_like(chi), torch.zeros_like(chi)
    ray = torch.arange(nx * ny, device="cuda")
    x0, y0 = ray % nx, ray // nx
    for di, dj, kk, s, n_pts, wmu, mu in _box_batches(case):
        def vox(m):
            y = (y0[None] + dj[:, m:m + 1]) % ny
            return (kk[:, m:m + 1] * ny + y) * nx + (x0[None] + di[:, m:m + 1]) % nx

        def at(m):
            v = vox(m)
            return chi[:, v], S[:, v], s[:, m:m + 1]

        def deposit(m, active, I, term):
            w = (wmu[:, None] * s[:, m:m + 1] * active).expand(-1, nx * ny)
            v = vox(m).reshape(-1)
            J.index_add_(1, v, (w * I).reshape(lam, -1))
            L.index_add_(1, v, (w * term).reshape(lam, -1))

        I0 = torch.where(mu[None, :] < 0.0, bc[:, :1], bc[:, 1:2])[:, :, None]
        _sweep(s.shape[1], at, n_pts[:, None], I0, case.get("lstar") == "parabolic", deposit)
    return J.reshape(lam, nz, ny, nx), L.reshape(lam, nz, ny, nx)


def _exact_box_step(case, seed):
    """The first step from J = B: J and S after one operator-splitting update, and Lambda*."""
    chi, eps, B, _, bc = (x.double() for x in _box_fields(case, seed))
    J_fs, L = _box_operator(case, chi, (1.0 - eps) * B + eps * B, bc)
    J = B + (J_fs - B) / (1.0 - (1.0 - eps) * L).clamp(min=1e-7 if case["prec"] == "f32" else 1e-12)
    return dict(J=J, S=(1.0 - eps) * J + eps * B, lstar=L)


def _exact_box_stencil(case, seed):
    nx, ny, nz, lam = case["nx"], case["ny"], case["nz"], case["lam"]
    n = nx * ny * nz
    parabolic = case["lstar"] == "parabolic"
    chi = _box_fields(case, seed)[0].double().reshape(lam, n)
    out = torch.zeros((lam, 27 * n), dtype=torch.float64, device="cuda")
    ray = torch.arange(nx * ny, device="cuda")
    x0, y0 = ray % nx, ray // nx
    for di, dj, kk, s, n_pts, wmu, _ in _box_batches(case):
        M = s.shape[1]

        def vox(m):
            y = (y0[None] + dj[:, m:m + 1]) % ny
            return (kk[:, m:m + 1] * ny + y) * nx + (x0[None] + di[:, m:m + 1]) % nx

        def depth(m):
            return chi[:, vox(m)] * s[:, m:m + 1]

        t = depth(0)
        tn = depth(min(1, M - 1))
        tp = t
        G = [torch.zeros_like(t) for _ in range(5)]  # dI/dS of the points m+1, m, m-1, m-2, m-3
        for m in range(M):
            if m == 0:
                G[1] = _moments(torch.clamp(0.5 * t, min=1e-100))[1]
            else:
                last = (n_pts <= m + 1)[:, None].expand_as(t)
                if parabolic:
                    ex, a, b, g, _ = _weights(0.5 * (tp + t), 0.5 * (t + tn), last)
                else:
                    D = torch.clamp(0.5 * (tp + t), min=1e-100)
                    ex, e0, e1, _ = _moments(D)
                    b = e1 / D
                    a, g = e0 - b, torch.zeros_like(b)
                G = [g, ex * G[0] + b, ex * G[1] + a, ex * G[2], ex * G[3]]
            v = vox(m)
            for j in range(-1, 4):
                u = m - j
                if u < 0 or u >= M:
                    continue
                d = [q[:, u] - q[:, m] for q in (di, dj, kk)]
                near = (n_pts > m) & (n_pts > u)
                for q in d:
                    near = near & (q.abs() <= 1)
                comp = torch.where(near, (d[2] + 1) * 9 + (d[1] + 1) * 3 + d[0] + 1, torch.zeros_like(d[0]))
                w = (wmu * s[:, m] * near)[:, None]
                out.index_add_(1, (comp[:, None] * n + v).reshape(-1), (w * G[j + 1]).reshape(lam, -1))
            tp, t = t, tn
            if m + 2 < M:
                tn = depth(m + 2)
    return out.reshape(lam, 27, nz, ny, nx)


class _Shell:
    """Characteristics of one direction on the shell 1 < r < 2: lattice lines, then one through every voxel missed."""

    def __init__(self, case):
        self.nr, self.nt, self.np = case["nr"], case["nt"], case["np"]
        r, c = 1.0 + np.arange(self.nr + 1) / self.nr, np.cos(np.arange(self.nt + 1) * math.pi / self.nt)
        vol = np.diff(r ** 3)[:, None] / 3.0 * -np.diff(c)[None, :] * (2.0 * math.pi / self.np)
        self.h = float(np.median(np.cbrt(vol)))

    def crossings(self, p, n):
        """Sorted crossing parameters (inf: none) of the lines p + t n with every voxel boundary."""
        pp = (p * p).sum(1, keepdims=True)
        inf = np.inf
        out = []
        with np.errstate(invalid="ignore", divide="ignore"):
            w = np.sqrt((1.0 + np.arange(1, self.nr) / self.nr)[None, :] ** 2 - pp)
            out += [-w, w]
            for k in range(1, self.nt):
                if 2 * k == self.nt:
                    out.append(-p[:, 2:3] / n[2])
                    continue
                c = math.cos(k * math.pi / self.nt)
                A, B, C = n[2] ** 2 - c * c, 2.0 * p[:, 2:3] * n[2], p[:, 2:3] ** 2 - c * c * pp
                q = np.sqrt(B * B - 4.0 * A * C)
                for t in ((-B - q) / (2.0 * A), (-B + q) / (2.0 * A)):
                    out.append(np.where((p[:, 2:3] + t * n[2] > 0.0) == (c > 0.0), t, inf))
            ph = 2.0 * math.pi * np.arange(self.np) / self.np
            cs, sn = np.cos(ph)[None, :], np.sin(ph)[None, :]
            t = (sn * p[:, :1] - cs * p[:, 1:2]) / (-sn * n[0] + cs * n[1])
            out.append(np.where(cs * (p[:, :1] + t * n[0]) + sn * (p[:, 1:2] + t * n[1]) > 0.0, t, inf))
        t = np.concatenate(out, axis=1)
        t[~np.isfinite(t)] = inf
        t.sort(axis=1)
        return t

    def locate(self, x):
        r = np.sqrt((x * x).sum(-1))
        th, ph = np.arccos(np.clip(x[..., 2] / r, -1.0, 1.0)), np.arctan2(x[..., 1], x[..., 0])
        ph = np.where(ph < 0.0, ph + 2.0 * math.pi, ph)
        idx = [np.clip(np.floor(v * m), 0, m - 1).astype(np.int64)
               for v, m in ((r - 1.0, self.nr), (th / math.pi, self.nt), (ph / (2.0 * math.pi), self.np))]
        return (idx[2] * self.nt + idx[1]) * self.nr + idx[0]

    def trace(self, p, n):
        """Padded (voxel, s) and count of visits, entry point and kind (1: starts on the core) per characteristic,
        with the index of its line."""
        pp = (p * p).sum(1)
        to, core = np.sqrt(4.0 - pp), pp < 1.0
        ti = np.sqrt(np.maximum(1.0 - pp, 0.0))
        idx = np.arange(len(p))
        line = np.concatenate([idx, idx[core]])
        ta = np.concatenate([-to, ti[core]])
        tb = np.concatenate([np.where(core, -ti, to), to[core]])
        kind = np.concatenate([np.zeros(len(p), int), np.ones(int(core.sum()), int)])
        order = np.argsort(2 * line + kind, kind="stable")
        line, ta, tb, kind = line[order], ta[order], tb[order], kind[order]
        t = self.crossings(p, n)[line]
        t = np.where((t > ta[:, None]) & (t < tb[:, None]), t, np.inf)
        t = np.concatenate([t, tb[:, None]], axis=1)
        t.sort(axis=1)
        t = t[:, :max(1, int(np.isfinite(t).sum(1).max()))]
        prev, keep, begin = ta.copy(), np.zeros(t.shape, bool), np.zeros(t.shape)
        for c in range(t.shape[1]):
            ok = np.isfinite(t[:, c]) & (t[:, c] - prev > 1e-12 * (np.abs(prev) + 1.0))
            keep[:, c], begin[:, c] = ok, prev
            prev = np.where(ok, t[:, c], prev)
        cnt = keep.sum(1)
        pos = np.argsort(~keep, axis=1, kind="stable")[:, :cnt.max()]
        b, e = np.take_along_axis(begin, pos, 1), np.take_along_axis(t, pos, 1)
        pad = np.arange(b.shape[1])[None, :] >= cnt[:, None]
        b, e = np.where(pad, ta[:, None], b), np.where(pad, ta[:, None], e)
        mid = 0.5 * (b + e)
        vox = self.locate(p[line][:, None, :] + mid[..., None] * np.asarray(n)[None, None, :])
        return np.where(pad, 0, vox), np.where(pad, 0.0, e - b), cnt, p[line] + ta[:, None] * np.asarray(n), kind, line

    def direction(self, n):
        """All characteristics of one direction: (vox, s, cnt, entry, kind)."""
        e1 = np.array([-n[1], n[0], 0.0])
        e1 = e1 / np.linalg.norm(e1) if np.linalg.norm(e1) >= 1e-12 else np.array([1.0, 0.0, 0.0])
        e2 = np.cross(n, e1)
        K = int(math.ceil(2.0 / self.h)) + 1
        a = np.arange(-K, K + 1)
        p = (a[:, None, None] * self.h * e1 + a[None, :, None] * self.h * e2).reshape(-1, 3)
        parts = [self.trace(p[(p * p).sum(1) < 4.0], n)[:5]]
        seen = np.zeros(self.nr * self.nt * self.np, bool)
        vox, _, cnt = parts[0][:3]
        seen[vox[np.arange(vox.shape[1])[None, :] < cnt[:, None]]] = True
        missed = np.nonzero(~seen)[0]
        if len(missed):
            ir, q = missed % self.nr, missed // self.nr
            r, th, ph = 1.0 + (ir + 0.5) / self.nr, (q % self.nt + 0.5) * math.pi / self.nt, \
                (q // self.nt + 0.5) * 2.0 * math.pi / self.np
            c = np.stack([r * np.sin(th) * np.cos(ph), r * np.sin(th) * np.sin(ph), r * np.cos(th)], axis=1)
            p = c - (c @ np.asarray(n))[:, None] * np.asarray(n)[None, :]
            full = self.trace(p, n)
            first = np.searchsorted(full[5], np.arange(len(p) + 1))
            used = np.zeros(len(full[5]), bool)
            for i, v in enumerate(missed):  # in voxel order, one line through every voxel still missed
                if seen[v]:
                    continue
                for c in range(first[i], first[i + 1]):
                    used[c] = True
                    seen[full[0][c, :full[2][c]]] = True
            parts.append(tuple(x[used] for x in full[:5]))
        M = max(x[0].shape[1] for x in parts)
        grow = [np.concatenate([np.pad(x[i], ((0, 0), (0, M - x[i].shape[1]))) for x in parts]) for i in (0, 1)]
        return (*grow, *(np.concatenate([x[i] for x in parts]) for i in (2, 3, 4)))


def _exact_sphere_fs(case, seed):
    lam, n_mu, n_phi = case["lam"], case["n_mu"], case["n_phi"]
    chi, S, bc = (x.double() for x in _sphere_fields(case, seed))
    shape = chi.shape
    chi, S = chi.reshape(lam, -1), S.reshape(lam, -1)
    J, L = torch.zeros_like(chi), torch.zeros_like(chi)
    ns = np.array([_direction(i, j, n_mu, n_phi) for i in range(n_mu) for j in range(n_phi)])
    shell, src, w = _Shell(case), np.array([0.0, 0.0, 10.0]), 1.0 / len(ns)
    for d, n in enumerate(ns):
        vox, s, cnt, entry, kind = shell.direction(n)
        u = entry - src
        dist = np.linalg.norm(u, axis=1)
        u = u / dist[:, None]
        lit = ((u * entry).sum(1) < 0.0) & (np.argmax(u @ ns.T, axis=1) == d) & (kind == 0)
        I_src = np.where(lit, 8.0 ** 2 / dist ** 2 / w, 0.0)
        if case["prec"] == "f32":  # the geometry of a single-precision grid
            weight_s, s = s, s.astype(np.float32).astype(np.float64)
        else:
            weight_s = s
        vox, s, weight_s, cnt, kind, I_src = (torch.from_numpy(np.ascontiguousarray(x)).cuda()
                                              for x in (vox, s, weight_s, cnt, kind, I_src))
        path = torch.zeros(chi.shape[1], dtype=torch.float64, device="cuda")
        path.index_add_(0, vox.reshape(-1), weight_s.reshape(-1))
        I0 = torch.where(kind[None] == 1, bc[:, 1:2], bc[:, :1] + bc[:, 2:3] * I_src[None])

        def at(m):
            return chi[:, vox[:, m]], S[:, vox[:, m]], s[:, m]

        def deposit(m, active, I, term):
            v = vox[:, m]
            k = w * weight_s[:, m] / path[v] * active
            J.index_add_(1, v, k * I)
            L.index_add_(1, v, k * term)

        _sweep(vox.shape[1], at, cnt, I0, case["lstar"] == "parabolic", deposit)
    return J.reshape(shape), L.reshape(shape)


def _exact_net(case, seed):
    """The network in 64 bits: periodic x and y, zero-padded z."""
    layers = iter(_net_layers(case, seed))
    L = len(_net_channels(case))

    def conv(x, stride=1, relu=True):
        taps, _, co, w, b = next(layers)
        w, b = torch.from_numpy(w).cuda().double(), torch.from_numpy(b).cuda().double()
        nz, ny, nx, _ = x.shape
        if taps == 1:
            return x @ w[0].t() + b
        iz, iy, ix = (torch.arange(0, m, stride, device="cuda") for m in (nz, ny, nx))
        y = b.expand(len(iz), len(iy), len(ix), co).clone()
        for t in range(27):
            z, yy, xx = iz + t // 9 - 1, (iy + (t // 3) % 3 - 1) % ny, (ix + t % 3 - 1) % nx
            ok = (z >= 0) & (z < nz)
            y[ok] += x[z[ok]][:, yy][:, :, xx] @ w[t].t()
        return y.relu() if relu else y

    def upsample(x, shape):
        for axis, n in enumerate(shape):
            o = torch.arange(n, device="cuda")
            hi = (o + 1) // 2
            hi = hi.clamp(max=x.shape[axis] - 1) if axis == 0 else hi % x.shape[axis]
            x = 0.5 * (x.index_select(axis, o // 2) + x.index_select(axis, hi))
        return x

    h = [conv(conv(_net_features(case, seed).double()))]
    for _ in range(1, L):
        h.append(conv(conv(h[-1], stride=2)))
    for k in range(L - 1, 0, -1):
        h[k - 1] = conv(conv(upsample(h[k], h[k - 1].shape[:3])) + h[k - 1])
    return conv(h[0], relu=False)[..., 0]


def exact(case, seed):
    kind = case["kind"]
    if kind == "net":
        return _exact_net(case, seed)
    if kind == "box_solve" or _points(case) > MAX_EXACT_POINTS:
        return None
    if kind == "box_step":
        return _exact_box_step(case, seed)
    if kind == "box_stencil":
        return _exact_box_stencil(case, seed)
    J, L = _exact_box_fs(case, seed) if kind == "box_fs" else _exact_sphere_fs(case, seed)
    return dict(J=J, lstar=L) if case["lstar"] != "none" else dict(J=J)
