"""Timed cases of the library: what a mock-making program has it do, over the
range it is used in, through the public binding.

A case is a dict of plain values with a "kind":

  box        one Gaussian box (make_box, or make_eta for other components)
  skewers    pixels along lines of sight through a box (trilinear, wide-angle
             or the 7^3 Gaussian kernel), with or without FGPA and bins
  post       post-production of stored pixels: delta_S redrawn (or not), FGPA
             and mean flux, then the 1D power
  labels     training labels of the tuning emulator
  train      loss and gradient of one training batch of the emulator
  quasars    variances of the quasar boxes, then the three-box quasar draw
  lognormal  the lognormal quasar spectrum P_q(k) and xi_m(r)

Boxes above 1024^3 are made by the benchmark, not here: their outputs and the
copies a comparison needs do not fit the card.  Reading one (skewers) does.

Inputs come from torch and numpy alone (never from the library), so that they
are the same whatever the library does; exact() evaluates the same quantities
in 64 bits from their definitions.
"""
import ctypes
import math

import numpy as np
import torch

from paper_2310_18996_amd import lyamock as L

DEV = "cuda"
OMEGA_M = 0.3147
C_H0 = 2997.92458          # c / H0, Mpc/h
DX = 2.19                  # voxel side, Mpc/h
DPIX = 0.2                 # pixel length, Mpc/h
LYA_A = 1215.67
PK = dict(sigma8=0.8, ns=0.96, gamma=0.21, wig_amp=0.05, wig_r=105.0, wig_kd=0.2)
Z_EDGES = np.round(np.linspace(1.6, 3.8, 23), 10)
PS_AMP, PS_KCUT = 1.0, 1.5
# P1D bins: 32 between 0.001 and 0.05 s/km, logarithmic
K_EDGES = 0.001 * 50.0 ** (np.arange(33) / 32.0)
# three quasar boxes and the k, r nodes of the lognormal transforms
QSO_Z = (1.9, 2.75, 3.6)


def _quad(c0, c1, c2, x0=3.5):
    """Powers of (1+z) of c0 + c1 x + c2 x^2 in x = (1+z) - x0."""
    return [c0 - c1 * x0 + c2 * x0 * x0, c1 - 2.0 * c2 * x0, c2]


FGPA = [_quad(0.5, 0.4, 0.1), _quad(1.6, -0.1, 0.0), _quad(1.535, -1.018, 0.483)]


# ------------------------------------------------------------------ the cases
def listed():
    return [
        # the smallest box (tests, examples, smoke runs): launches and tables count
        dict(name="box_64", kind="box", n=64, storage="f32", comps="delta,zz", two_buffer=True),
        # velocity pair of the quasar catalogue on the 512^3 mock, in place
        dict(name="box_512_velocity", kind="box", n=512, storage="f32", comps="vx,vy", two_buffer=False),
        # the 1024^3 precision configuration in BF16 storage, default workspace
        dict(name="box_1024_bf16", kind="box", n=1024, storage="bf16", comps="delta,zz", two_buffer=False),
        # 500 skewers of 256 pixels on the 64^3 box: the smallest pass
        dict(name="skewers_64", kind="skewers", n=64, storage="f32", n_sk=500, npix_min=256, npix_max=256,
             interp="tri", geometry="box", fgpa=True, bins=False),
        # the largest pass: 1M uneven skewers (200-2000 pixels) through a 2048^3 box, FGPA and 22 bins fused
        dict(name="skewers_2048", kind="skewers", n=2048, storage="f32", n_sk=1000000, npix_min=200, npix_max=2000,
             interp="tri", geometry="radial", fgpa=True, bins=True),
        # wide-angle eta_par from four BF16 boxes, odd skewer count
        dict(name="wide_512_bf16", kind="skewers", n=512, storage="bf16", n_sk=50001, npix_min=200, npix_max=1200,
             interp="wide", geometry="radial", fgpa=True, bins=True),
        # the paper's 7^3 Gaussian kernel before FGPA (its make_spectra step) on the 512^3 mock
        dict(name="gauss_512", kind="skewers", n=512, storage="f32", n_sk=50000, npix_min=200, npix_max=1200,
             interp="gauss", geometry="radial", fgpa=False, bins=False),
        # post-production on the pixels of the 512^3 mock, as each P_s iteration runs it
        dict(name="post_50k", kind="post", n_sk=50000, npix_min=200, npix_max=1200, delta_s=True),
        # emulator labels on the pixels of the 256^3 mock
        dict(name="labels_20k", kind="labels", n_sk=20000, npix_min=200, npix_max=1200, draws=64, delta_s=False),
        # one training batch of the tuning emulator
        dict(name="train_512", kind="train", batch=512, n_out=33, bf16=True),
        # quasar draw from three 1024^3 lognormal boxes
        dict(name="quasars_1024", kind="quasars", n=1024, density=1e-5),
        # one box's lognormal spectrum with the transform's full r and k ranges
        dict(name="lognormal", kind="lognormal", n_r=40001, n_k=512, rmax=2000.0, smooth=DX),
    ]


def _logint(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["box", "box", "skewers", "skewers", "skewers", "post", "labels", "train", "quasars",
                       "lognormal"])
    storage = rng.choice(["f32", "bf16"])
    if kind == "box":
        return dict(kind=kind, n=rng.choice([64, 128, 256, 512, 1024]), storage=storage,
                    comps=rng.choice(["delta,zz", "delta,none", "xx,yy", "xy,xz", "vx,vy", "vz,none"]),
                    two_buffer=rng.random() < 0.5)
    lo = rng.randint(20, 400)
    hi = lo + rng.randint(0, 1600)
    if kind == "skewers":
        interp = rng.choice(["tri", "tri", "wide", "gauss"])
        fgpa = rng.random() < 0.7
        return dict(kind=kind, n=rng.choice([64, 128, 256, 512, 1024]), storage=storage,
                    n_sk=_logint(rng, 300, 60000 if interp == "gauss" else 200000), npix_min=lo, npix_max=hi,
                    interp=interp, geometry=rng.choice(["radial", "radial", "box"]), fgpa=fgpa,
                    bins=fgpa and rng.random() < 0.7)
    if kind == "post":
        return dict(kind=kind, n_sk=_logint(rng, 300, 100000), npix_min=lo, npix_max=hi,
                    delta_s=rng.random() < 0.5)
    if kind == "labels":
        return dict(kind=kind, n_sk=_logint(rng, 300, 20000), npix_min=lo, npix_max=hi, draws=_logint(rng, 1, 48),
                    delta_s=rng.random() < 0.3)
    if kind == "train":
        return dict(kind=kind, batch=_logint(rng, 32, 2048), n_out=rng.randint(5, 64), bf16=rng.random() < 0.75)
    if kind == "quasars":
        return dict(kind=kind, n=rng.choice([128, 256, 512]), density=round(rng.uniform(0.5, 3.0), 3) * 1e-5)
    return dict(kind=kind, n_r=2 * _logint(rng, 1000, 20000) + 1, n_k=_logint(rng, 64, 700),
                rmax=round(rng.uniform(500.0, 2000.0), 1), smooth=round(rng.uniform(2.0, 5.0), 3))


# ------------------------------------------------------------------ inputs
def _gen(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(int(seed) + 77)
    return g


def _chi(z):
    """Comoving distance (Mpc/h), numpy Gauss-Legendre, 64 bits."""
    z = np.atleast_1d(np.asarray(z, dtype=np.float64))
    x, w = np.polynomial.legendre.leggauss(48)
    t = 0.5 * z[:, None] * (x[None, :] + 1.0)
    return C_H0 * 0.5 * z * np.sum(w / np.sqrt(OMEGA_M * (1.0 + t) ** 3 + 1.0 - OMEGA_M), axis=1)


_TABLE = {}


def _chi_table():
    """(z, chi) nodes on the GPU for placing quasars."""
    if "t" not in _TABLE:
        z = np.linspace(0.0, 5.0, 4001)
        _TABLE["t"] = (torch.from_numpy(z).to(DEV), torch.from_numpy(_chi(z)).to(DEV))
    return _TABLE["t"]


def _chi_gpu(z):
    zt, ct = _chi_table()
    t = z / (zt[1] - zt[0])
    i = t.floor().clamp(0, zt.numel() - 2).long()
    return ct[i] + (t - i) * (ct[i + 1] - ct[i])


def _skewer_table(case, g):
    """The skewer table (GPU tensors): radial lines within 5 degrees of z from an
    observer at z = 2.5 below the box, lengths affine in the quasar's redshift
    (1.8-3.6, evenly spread, so that every seed has as many pixels), longest
    first; or origins anywhere in the box."""
    s, n = case["n_sk"], case.get("n", 512)
    side = n * DX
    obs = torch.tensor([side / 2, side / 2, -float(_chi(2.5)[0])], dtype=torch.float64, device=DEV)
    frac = (torch.arange(s, dtype=torch.float64, device=DEV) + 0.5) / s
    if case.get("geometry", "radial") == "box":
        x0 = torch.rand((s, 3), generator=g, dtype=torch.float64, device=DEV) * side
        d = x0 - obs
        chi0 = d.norm(dim=1)
        u = d / chi0[:, None]
    else:
        cos_t = 1.0 - (1.0 - math.cos(math.radians(5.0))) * torch.rand(s, generator=g, dtype=torch.float64, device=DEV)
        phi = 2 * math.pi * torch.rand(s, generator=g, dtype=torch.float64, device=DEV)
        sin_t = (1.0 - cos_t * cos_t).clamp(min=0.0).sqrt()
        u = torch.stack([sin_t * phi.cos(), sin_t * phi.sin(), cos_t], dim=1)
        chi0 = _chi_gpu((2.8 + 1.8 * frac) * (1200.0 / LYA_A) - 1.0)
        x0 = obs + chi0[:, None] * u
    npix = (case["npix_min"] + (case["npix_max"] - case["npix_min"]) * frac).round().to(torch.int32)
    order = torch.argsort(npix, descending=True, stable=True)
    x0, u, chi0, npix = x0[order], u[order], chi0[order].contiguous(), npix[order].contiguous()
    off = torch.zeros(s, dtype=torch.int64, device=DEV)
    off[1:] = torch.cumsum(npix[:-1].long(), 0)
    two32 = 2.0 ** 32
    return dict(origin=(x0 / DX * two32).round().long().contiguous(),
                step=(u * (-DPIX / DX) * two32).round().long().contiguous(), npix=npix, off=off, chi0=chi0,
                total=int(npix.long().sum()))


def _struct(t):
    return L.skewers_struct(t["npix"].numel(), t.get("origin"), t.get("step"), t["npix"], t["off"], t["chi0"], DPIX)


def _field(case, g, sigma):
    """A box of independent normals (sigma of the two components)."""
    n = case["n"]
    elems = n * (n * n + 32)
    if case.get("storage", "f32") == "bf16":
        f = torch.empty((elems, 2), dtype=torch.bfloat16, device=DEV)
        f.normal_(generator=g)
        f[:, 0] *= sigma[0]
        f[:, 1] *= sigma[1]
        return f.view(torch.int32).view(-1)
    f = torch.empty((elems, 2), dtype=torch.float32, device=DEV)
    f.normal_(generator=g)
    f[:, 0] *= sigma[0]
    f[:, 1] *= sigma[1]
    return f


def _bins(s):
    edges = torch.from_numpy(_chi(Z_EDGES)).to(DEV)
    s["edges"] = edges
    s["fsum"] = torch.zeros(len(Z_EDGES) - 1, dtype=torch.float64, device=DEV)
    s["count"] = torch.zeros(len(Z_EDGES) - 1, dtype=torch.int64, device=DEV)
    s["zb"] = L.zbins_struct(edges, s["fsum"], s["count"])


def _pixels(total, g):
    """Stored pixels: delta_L and eta_par correlated over a voxel (11 pixels)."""
    out = []
    for sigma in (1.6, 0.8):
        x = torch.randn(total + 20, generator=g, dtype=torch.float32, device=DEV)
        x = torch.nn.functional.avg_pool1d(x.view(1, 1, -1), 11, stride=1).view(-1)[:total]
        out.append((x * (sigma * math.sqrt(11.0))).contiguous())
    return out


def _f32(x):
    return torch.empty(x, dtype=torch.float32, device=DEV)


def _bytes(x):
    return torch.empty(x, dtype=torch.uint8, device=DEV)


def prepare(case, seed):
    kind, s = case["kind"], dict(case=case, seed=int(seed) * 2 + 1)
    if kind == "box":
        n = case["n"]
        bf = case["storage"] == "bf16"
        s["box"] = L.box_struct(n, DX, L.LYA_BF16 if bf else L.LYA_F32)
        s["pk"] = L.pk_struct(**PK)
        op = L.LYA_OP_BOX_2BUF if case["two_buffer"] else L.LYA_OP_BOX
        s["work"] = _bytes(L.workspace_size(op, s["box"]))
        e = L.field_elems(s["box"])
        s["field"] = torch.empty(e, dtype=torch.int32, device=DEV) if bf else _f32((e, 2))
        return s
    g = _gen(seed)
    if kind == "skewers":
        bf = case["storage"] == "bf16"
        s["box"] = L.box_struct(case["n"], DX, L.LYA_BF16 if bf else L.LYA_F32)
        s["t"] = _skewer_table(case, g)
        s["sk"] = _struct(s["t"])
        s["fields"] = [_field(case, g, (1.6, 0.8))]
        if case["interp"] == "wide":
            s["fields"] += [_field(case, g, (0.5, 0.5)) for _ in range(3)]
        s["ps"] = L.Ps1d(PS_AMP, PS_KCUT, DPIX, 0)
        s["cosmo"] = L.Cosmo(OMEGA_M)
        s["fgpa"] = L.fgpa_struct(FGPA) if case["fgpa"] else None
        s["dens"], s["eta"] = _f32(s["t"]["total"]), _f32(s["t"]["total"])
        s["flux"] = _f32(s["t"]["total"]) if case["fgpa"] else None
        s["zb"] = None
        if case["bins"]:
            _bins(s)
        s["work"] = _bytes(L.workspace_size(L.LYA_OP_SKEWERS))
        return s
    if kind in ("post", "labels"):
        s["t"] = _skewer_table(dict(case, n=512, geometry="radial"), g)
        s["sk"] = _struct(s["t"])
        s["dens"], s["eta"] = _pixels(s["t"]["total"], g)
        s["cosmo"] = L.Cosmo(OMEGA_M)
        s["k_edges"] = torch.from_numpy(K_EDGES).to(DEV)
        if kind == "post":
            s["fgpa"] = L.fgpa_struct(FGPA)
            s["flux"] = _f32(s["t"]["total"])
            _bins(s)
            s["ps"] = L.Ps1d(PS_AMP, PS_KCUT, DPIX, 0)
            # per-bin factors of P_s, as a few iterations leave them; bins of the P1D in h/Mpc at z = 2.5
            s["ps_k"] = s["k_edges"] * _km_s(2.5)
            s["ratio"] = torch.exp(0.3 * torch.randn(32, generator=g, dtype=torch.float32, device=DEV))
            s["table"] = L.PsTable(32, s["ps_k"].data_ptr(), s["ratio"].data_ptr())
            s["spec"] = L.P1dSpec(32, s["k_edges"].data_ptr(), 2.5, DPIX)
            s["psum"] = torch.zeros(32, dtype=torch.float64, device=DEV)
            s["pcount"] = torch.zeros(32, dtype=torch.int64, device=DEV)
            s["work"] = _bytes(L.workspace_size(L.LYA_OP_SKEWERS))
            s["pwork"] = _bytes(L.p1d_workspace_size(case["n_sk"], 32))
            return s
        rng = np.random.default_rng([int(seed), 5])
        k = case["draws"]
        if case["delta_s"]:   # (a, b, amp, kcut)
            s["draws"] = np.stack([rng.uniform(0.1, 1.0, k), rng.uniform(1.0, 2.2, k), rng.uniform(0.5, 2.0, k),
                                   rng.uniform(0.8, 2.0, k)], axis=1)
        else:                 # (a, b, c, z), a log-uniform
            s["draws"] = np.stack([np.exp(rng.uniform(math.log(1e-3), math.log(5.0), k)), rng.uniform(1.0, 2.2, k),
                                   rng.uniform(0.5, 2.6, k), rng.uniform(1.8, 3.6, k)], axis=1)
        s["y"] = _f32((k, 33))
        if case["delta_s"]:
            sp = L.TunePsSpec()
            sp.sk = ctypes.pointer(s["sk"])
            sp.dens_l, sp.eta = s["dens"].data_ptr(), s["eta"].data_ptr()
            sp.n_pixels, sp.cosmo, sp.seed, sp.n_zt = s["t"]["total"], s["cosmo"], s["seed"], 1
            sp.z_t[0], sp.c_t[0], sp.fbar_t[0] = 2.5, 1.2, 0.6
            s["p1d_t"] = np.ones((1, 32))
            sp.p1d_t = s["p1d_t"].ctypes.data
            sp.p1d = L.P1dSpec(32, s["k_edges"].data_ptr(), 0.0, DPIX)
            sp.ps_amp, sp.ps_kcut, sp.n_iter = PS_AMP, PS_KCUT, 1
            s["spec"] = sp
            s["work"] = _bytes(L.tune_ps_workspace_size(case["n_sk"], s["t"]["total"], 32))
        else:
            s["spec"], s["keep"] = L.tune_spec(s["sk"], s["dens"], s["eta"], s["cosmo"], [2.5], [1.0], [0.5],
                                               np.ones((1, 32)), s["k_edges"], DPIX)
            s["work"] = _bytes(L.tune_workspace_size(case["n_sk"], 32))
        return s
    if kind == "train":
        b, no = case["batch"], case["n_out"]
        emu = torch.zeros(L.emulator_bytes(no), dtype=torch.uint8, device=DEV)
        L.emulator_init(emu, no, 1, 1, [1e-3, 1.0, 0.5, 1.8], [5.0, 2.2, 2.6, 3.6], log_inputs=1)
        o = L.emulator_param_offset()
        p = emu[o:o + 4 * L.emulator_param_count(no)].view(torch.float32)
        p.normal_(generator=g)
        for (lo, hi, fan) in _layers(no):   # He-normal weights, small biases
            p[lo[0]:lo[1]] *= math.sqrt(2.0 / fan)
            p[hi[0]:hi[1]] *= 0.05
        s["emu"], s["params"] = emu, p
        s["x0"] = torch.rand((b, 4), generator=g, dtype=torch.float32, device=DEV) * 2.0 - 1.0
        s["tgt"] = torch.randn((b, no), generator=g, dtype=torch.float32, device=DEV)
        s["grad"], s["loss"] = _f32(p.numel()), _f32(1)
        s["work"] = _bytes(L.emulator_train_workspace_size(b, no))
        return s
    if kind == "quasars":
        n = case["n"]
        s["box"] = L.box_struct(n, DX)
        s["fields"] = [_field(case, g, (1.3, 1.2)), _field(case, g, (1.1, 0.0))]
        z = np.round(np.linspace(1.7, 4.0, 24), 10)
        shape = (1 + z) ** 2 * np.exp(-((z - 2.3) / 0.6) ** 2)
        s["nz"] = torch.from_numpy(z).to(DEV)
        s["nb"] = torch.from_numpy(case["density"] * shape / shape.max()).to(DEV)
        s["mom"] = torch.zeros(8, dtype=torch.float64, device=DEV)
        base = s["mom"].data_ptr()
        s["pos"] = torch.zeros((1 << 18, 3), dtype=torch.int64, device=DEV)
        s["cat"] = torch.zeros_like(s["pos"])
        s["cnt"] = torch.zeros(1, dtype=torch.int64, device=DEV)
        side = n * DX
        s["spec"] = L.qso_spec(s["fields"], QSO_Z, [base + 8, base + 24, base + 40],
                               [side / 2, side / 2, -float(_chi(1.8)[0])], s["nz"], s["nb"], s["seed"], 0.12)
        s["cosmo"] = L.Cosmo(OMEGA_M)
        s["work"] = _bytes(L.workspace_size(L.LYA_OP_QUASARS, s["box"]))
        return s
    # lognormal: the smoothing length and k nodes move a little with the seed
    rng = np.random.default_rng([int(seed), 9])
    s["sigma8"] = 0.8 * (1.0 + 0.02 * rng.uniform(-1, 1))
    s["pk"] = L.pk_struct(**dict(PK, sigma8=s["sigma8"]), smooth=case["smooth"])
    kk = np.geomspace(7e-4, 2.6, case["n_k"]) * (1.0 + 0.01 * rng.uniform(-1, 1))
    s["k"] = torch.from_numpy(kk).to(DEV)
    s["pq"] = torch.zeros(case["n_k"], dtype=torch.float64, device=DEV)
    s["xi"] = torch.zeros(case["n_r"], dtype=torch.float64, device=DEV)
    s["cosmo"] = L.Cosmo(OMEGA_M)
    s["work"] = _bytes(L.lognormal_workspace_size(case["smooth"], case["rmax"], case["n_r"]))
    return s


def _layers(no):
    """((weights lo, hi), (biases lo, hi), fan_in) of the emulator's parameters."""
    out, p = [], 0
    for fi, fo in ((4, 256), (256, 256), (256, 256), (256, no)):
        out.append(((p, p + fi * fo), (p + fi * fo, p + fi * fo + fo), fi))
        p += fi * fo + fo
    return out


def _km_s(z):
    """km/s per Mpc/h at z."""
    return 100.0 * math.sqrt(OMEGA_M * (1 + z) ** 3 + 1 - OMEGA_M) / (1 + z)


# ------------------------------------------------------------------ one pass
def run(s):
    case = s["case"]
    kind = case["kind"]
    if kind == "box":
        a, b = case["comps"].split(",")
        if a == "delta" and b in ("zz", "none"):
            L.make_box(s["box"], s["pk"], s["seed"], 1.0, b == "zz", s["field"], s["work"])
        else:
            L.make_eta(s["box"], s["pk"], s["seed"], 1.0, a, b, s["field"], s["work"])
        v = L.box_view(s["field"], case["n"])
        return v.view(torch.bfloat16) if case["storage"] == "bf16" else v
    if kind == "skewers":
        args = (s["sk"], s["ps"], s["seed"], s["cosmo"], s["fgpa"], s["dens"], s["eta"], s["flux"], s["zb"], s["work"])
        if case["interp"] == "wide":
            L.draw_skewers_wide(s["box"], s["fields"], *args)
        elif case["interp"] == "gauss":
            L.draw_skewers_gauss(s["box"], s["fields"][0], *args)
        else:
            L.draw_skewers(s["box"], s["fields"][0], *args)
        out = dict(dens=s["dens"], eta=s["eta"])
        if case["fgpa"]:
            out["flux"] = s["flux"]
        if case["bins"]:
            out["fsum"], out["count"] = s["fsum"], s["count"]
        return out
    if kind == "post":
        if case["delta_s"]:
            L.apply_fgpa_ds(s["sk"], s["cosmo"], s["dens"], s["eta"], s["ps"], s["table"], s["seed"], s["fgpa"],
                            s["flux"], s["zb"], s["work"])
        else:
            L.apply_fgpa(s["sk"], s["cosmo"], s["dens"], s["eta"], s["fgpa"], s["flux"], s["zb"], s["work"])
        L.p1d(s["sk"], s["cosmo"], s["flux"], s["zb"], s["spec"], s["psum"], s["pcount"], s["pwork"])
        return dict(flux=s["flux"], fsum=s["fsum"], count=s["count"], psum=s["psum"], pcount=s["pcount"])
    if kind == "labels":
        if case["delta_s"]:
            L.emulator_labels_ps(s["spec"], 0, s["draws"], s["y"], s["work"])
        else:
            L.emulator_labels(s["spec"], s["draws"], s["y"], s["work"])
        return s["y"]
    if kind == "train":
        L.emulator_loss_grad(s["emu"], s["x0"], s["tgt"], case["batch"], case["bf16"], s["grad"], s["loss"], s["work"])
        return dict(grad=s["grad"], loss=s["loss"])
    if kind == "quasars":
        L.box_moments(s["box"], s["fields"][0], s["mom"][:4], s["work"])
        L.box_moments(s["box"], s["fields"][1], s["mom"][4:], s["work"])
        L.draw_quasars(s["box"], s["spec"], s["cosmo"], s["pos"], s["cnt"], s["work"])
        # the catalogue by voxel, so that it is reproducible (the draw's order is unspecified)
        n = case["n"]
        c = min(int(s["cnt"].item()), s["pos"].shape[0])
        p = s["pos"][:c]
        m = (p + (1 << 31)) >> 32
        s["cat"].zero_()
        s["cat"][:c] = p[torch.argsort((m[:, 0] * n + m[:, 1]) * n + m[:, 2])]
        return dict(moments=s["mom"], count=s["cnt"], pos=s["cat"])
    L.lognormal_pk(s["pk"], QSO_Z[0], QSO_Z[1], s["cosmo"], case["rmax"], case["n_r"], s["k"], s["pq"], s["xi"],
                   s["work"])
    return dict(pq=s["pq"], xi=s["xi"])


# ------------------------------------------------------------------ work of a pass
def work(case):
    kind = case["kind"]
    if kind == "box":
        cells = float(case["n"]) ** 3
        return dict(bytes=cells * (4 if case["storage"] == "bf16" else 8), flops=5 * cells * 3 * math.log2(case["n"]))
    if kind in ("skewers", "post", "labels"):
        pix = case["n_sk"] * 0.5 * (case["npix_min"] + case["npix_max"])
        table = 68.0 * case["n_sk"]
    if kind == "skewers":
        cell = 4 if case["storage"] == "bf16" else 8
        boxes = 4 if case["interp"] == "wide" else 1
        # columns of voxels a line passes, one voxel per DX/DPIX pixels, at most the box itself
        cols = 49 if case["interp"] == "gauss" else 4
        vox = min(float(case["n"]) ** 3, cols * pix * DPIX / DX)
        out = 12 if case["fgpa"] else 8
        per = dict(tri=28, wide=28 + 16 * 8, gauss=4 * 343)[case["interp"]] + 5 * 10 + (40 if case["fgpa"] else 0)
        return dict(bytes=table + pix * out + vox * cell * boxes, flops=pix * per)
    if kind == "post":
        return dict(bytes=table + pix * 16, flops=pix * (40 + 25 + (50 if case["delta_s"] else 0)))
    if kind == "labels":
        return dict(bytes=table + pix * 8, flops=pix * case["draws"] * (30 + 25 + (50 if case["delta_s"] else 0)))
    if kind == "train":
        p = sum(h[1] - l[0] for l, h, _ in _layers(case["n_out"]))
        return dict(bytes=8.0 * p + 4.0 * case["batch"] * (4 + case["n_out"]), flops=6.0 * case["batch"] * p)
    if kind == "quasars":
        cells = float(case["n"]) ** 3
        return dict(bytes=16 * cells, flops=60 * cells)
    kmax = 12.0 / case["smooth"]
    m = kmax / min(0.1 / case["rmax"], kmax / 64.0)
    return dict(bytes=8.0 * (case["n_r"] + 2 * case["n_k"]), flops=2.0 * case["n_r"] * (m + case["n_k"]))


# ------------------------------------------------------------------ 64-bit values
M32 = 0xFFFFFFFF


def _mul(a, x):
    """(high, low) 32-bit words of a * x for 32-bit values in int64."""
    p, q = a * (x & 0xFFFF), a * (x >> 16)
    t = q + (p >> 16)
    return t >> 16, ((t & 0xFFFF) << 16) | (p & 0xFFFF)


def _philox(c0, c1, stream, seed):
    """Philox4x32-10 (Salmon et al. 2011) words of counters (c0, c1, stream, 0)."""
    k0, k1 = seed & M32, seed >> 32
    c2, c3 = torch.full_like(c0, stream), torch.zeros_like(c0)
    for _ in range(10):
        h0, l0 = _mul(0xD2511F53, c0)
        h1, l1 = _mul(0xCD9E8D57, c2)
        c0, c1, c2, c3 = h1 ^ c1 ^ k0, l1, h0 ^ c3 ^ k1, l0
        k0, k1 = (k0 + 0x9E3779B9) & M32, (k1 + 0xBB67AE85) & M32
    return c0, c1, c2, c3


def _normals(seed, stream, lin):
    """The Box-Muller pair of each linear index, 64 bits."""
    ctr = lin >> 1
    w = _philox(ctr & M32, ctr >> 32, stream, seed)
    odd = (lin & 1) == 1
    a, b = torch.where(odd, w[2], w[0]), torch.where(odd, w[3], w[1])
    u = ((a >> 9).double() + 0.5) * 2.0 ** -23
    t = ((b >> 9).double() + 0.5) * 2.0 ** -23
    r = torch.sqrt(-2.0 * torch.log(u))
    return r * torch.cos(2 * math.pi * t), r * torch.sin(2 * math.pi * t)


def _pk_shape(k):
    q = k / PK["gamma"]
    x = 2.34 * q
    t = np.log1p(x) / x * (1 + 3.89 * q + (16.1 * q) ** 2 + (5.46 * q) ** 3 + (6.71 * q) ** 4) ** -0.25
    return k ** PK["ns"] * t * t * (1 + PK["wig_amp"] * np.sin(k * PK["wig_r"]) * np.exp(-(k / PK["wig_kd"]) ** 2))


def _pk_amp(sigma8):
    lk = np.linspace(math.log(1e-5), math.log(1e3), 65537)
    k = np.exp(lk)
    x = 8.0 * k
    small = x < 1e-2
    xs = np.where(small, 1.0, x)
    w = np.where(small, 1 - x * x / 10 + x ** 4 / 280, 3 * (np.sin(xs) - xs * np.cos(xs)) / xs ** 3)
    wt = np.full(65537, 2.0)
    wt[1::2] = 4.0
    wt[0] = wt[-1] = 1.0
    s = np.sum(wt * k ** 3 * _pk_shape(k) * w * w) * (lk[1] - lk[0]) / 3.0 / (2 * math.pi ** 2)
    return sigma8 ** 2 / s


def _exact_box(case, seed):
    n = case["n"]
    side = n * DX
    e = np.arange(1, 3 * (n // 2) ** 2 + 1, dtype=np.float64)
    tab = np.concatenate([[0.0], np.sqrt(_pk_amp(PK["sigma8"]) * _pk_shape(2 * math.pi * np.sqrt(e) / side) / side ** 3)])
    tab = torch.from_numpy(tab).to(DEV)
    i = torch.arange(n, device=DEV)
    f = torch.where(i < n // 2, i, i - n)
    x = torch.empty((n, n, n), dtype=torch.complex128, device=DEV)
    comps = case["comps"].split(",")
    step = max(1, (1 << 23) // (n * n))

    def mult(c, fr, n2):
        """Multiplier of delta_hat: (value, whether it is imaginary)."""
        inv = torch.where(n2 > 0, 1.0 / n2.clamp(min=1).double(), 0.0)
        if c[0] == "v":
            k = fr["xyz".index(c[1])]
            return torch.where(k == -(n // 2), 0.0, 100.0 * side / (2 * math.pi) * k.double() * inv), True
        p, q = fr["xyz".index(c[0])], fr["xyz".index(c[1])]
        v = (p * q).double() * inv
        return (torch.where((p == -(n // 2)) | (q == -(n // 2)), 0.0, v) if c[0] != c[1] else v), False

    for x0 in range(0, n, step):
        gx, gy, gz = torch.meshgrid(i[x0:x0 + step], i, i, indexing="ij")
        lin = (gx * n + gy) * n + gz
        plin = (((n - gx) % n) * n + (n - gy) % n) * n + (n - gz) % n
        z1, z2 = _normals(seed, 0, torch.minimum(lin, plin))
        h = math.sqrt(0.5)
        w = torch.complex(torch.where(lin == plin, z1, h * z1),
                          torch.where(lin == plin, 0.0, torch.where(lin > plin, -h * z2, h * z2)))
        fr = (f[gx], f[gy], f[gz])
        n2 = fr[0] ** 2 + fr[1] ** 2 + fr[2] ** 2
        w = w * tab[n2]
        acc = torch.zeros_like(w)
        for k, c in enumerate(comps):
            if c == "none":
                continue
            v = w
            if c != "delta":
                m, imag = mult(c, fr, n2)
                v = w * m * (1j if imag else 1.0)
            acc = acc + (v if k == 0 else 1j * v)
        x[x0:x0 + step] = acc
    del acc, w, v
    y = torch.fft.ifftn(x, norm="forward")
    del x
    out = torch.view_as_real(y)
    if comps[1] == "none":
        out[..., 1] = 0.0
    return out.reshape(n, n, 2 * n) if case["storage"] == "bf16" else out


def _z_of_chi(chi):
    """Redshift of a comoving distance: cubic Hermite between nodes (dz/dchi = E H0/c)."""
    if "h" not in _TABLE:
        step = 0.5
        c = np.arange(0.0, 6501.0, step)
        z = c / C_H0
        for _ in range(12):
            z = z - (_chi(z) - c) * np.sqrt(OMEGA_M * (1 + z) ** 3 + 1 - OMEGA_M) / C_H0
        d = np.sqrt(OMEGA_M * (1 + z) ** 3 + 1 - OMEGA_M) / C_H0
        _TABLE["h"] = (step, torch.from_numpy(z).to(DEV), torch.from_numpy(d).to(DEV))
    step, z, d = _TABLE["h"]
    i = (chi / step).floor().clamp(0, z.numel() - 2).long()
    t = chi / step - i
    z0, z1, d0, d1 = z[i], z[i + 1], d[i] * step, d[i + 1] * step
    return z0 + t * (d0 + t * (3 * (z1 - z0) - 2 * d0 - d1 + t * (2 * (z0 - z1) + d0 + d1)))


def _groups(npix, size_of, limit):
    """Runs of skewers [q0, q1) with the same size_of(npix) and size * count <= limit."""
    sizes = [size_of(int(v)) for v in npix]
    q = 0
    while q < len(sizes):
        e = q
        most = max(1, limit // max(1, sizes[q]))
        while e < len(sizes) and sizes[e] == sizes[q] and e - q < most:
            e += 1
        yield q, e, sizes[q]
        q = e


def _pow2_up(v):
    return 1 << max(0, (v - 1).bit_length()) if v > 1 else 1


def _normals_ds(seed, q0, q1, ns):
    m = torch.arange(ns // 2 + 1, device=DEV)
    return _normals(seed, 1, (torch.arange(q0, q1, device=DEV)[:, None] << 33) + m)


def _delta_s(zz, ns, amp, kcut, table=None):
    """delta_S of lines of ns pixels (rows) from their normal pairs."""
    m = torch.arange(ns // 2 + 1, device=DEV)
    k = 2 * math.pi * m.double() / (ns * DPIX)
    p = amp * torch.exp(-(k / kcut) ** 2)
    if table is not None:
        edges, ratio = table
        p = p * ratio[(torch.searchsorted(edges, k, right=True) - 1).clamp(0, ratio.numel() - 1)]
    a = torch.sqrt(p / (ns * DPIX))
    a[0] = 0.0
    w = torch.complex(zz[0] * math.sqrt(0.5), zz[1] * math.sqrt(0.5))
    w[:, -1] = torch.complex(zz[0][:, -1], torch.zeros_like(zz[0][:, -1]))
    return torch.fft.irfft(w * a, n=ns) * ns


def _exact_skewers(case, seed):
    st = prepare(case, seed)
    t, n = st["t"], case["n"]
    fields = [f.view(torch.bfloat16).view(-1, 2) if case["storage"] == "bf16" else f for f in st["fields"]]
    pitch = n * n + 32
    out = {k: torch.zeros(t["total"], dtype=torch.float64, device=DEV)
           for k in ("dens", "eta") + (("flux",) if case["fgpa"] else ())}
    co = FGPA
    edges = st.get("edges")
    fsum = torch.zeros(len(Z_EDGES) - 1, dtype=torch.float64, device=DEV)

    def comp(idx, k, c):
        return fields[k][idx, c].double()

    def interpolate(pos, u):
        """delta and eta_par at fixed-point positions [P, 3]; u: directions [P, 3]."""
        if case["interp"] == "gauss":
            cell = (pos + (1 << 31)) >> 32
            fr = (pos - (cell << 32)).double() / 2.0 ** 32
            o = torch.arange(-3, 4, device=DEV)
            g = torch.exp(-0.5 * (o[None, None, :] - fr[:, :, None]) ** 2)
            g = g / g.sum(dim=2, keepdim=True)
            d = torch.zeros(pos.shape[0], dtype=torch.float64, device=DEV)
            e = torch.zeros_like(d)
            for i in range(7):
                for j in range(7):
                    row = ((cell[:, 0] + i - 3) % n) * pitch + ((cell[:, 1] + j - 3) % n) * n
                    wij = g[:, 0, i] * g[:, 1, j]
                    for k in range(7):
                        v = fields[0][row + (cell[:, 2] + k - 3) % n].double()
                        w = wij * g[:, 2, k]
                        d += w * v[:, 0]
                        e += w * v[:, 1]
            return d, e
        cell = pos >> 32
        fr = (pos & M32).double() / 2.0 ** 32
        d = torch.zeros(pos.shape[0], dtype=torch.float64, device=DEV)
        e = torch.zeros_like(d)
        for c in range(8):
            b = torch.tensor([(c >> 2) & 1, (c >> 1) & 1, c & 1], device=DEV)
            w = torch.where(b == 1, fr, 1.0 - fr).prod(dim=1)
            i = (cell + b) % n
            idx = i[:, 0] * pitch + i[:, 1] * n + i[:, 2]
            v = fields[0][idx].double()
            d += w * v[:, 0]
            if case["interp"] == "tri":
                e += w * v[:, 1]
            else:
                v1, v2, v3 = (fields[k][idx].double() for k in (1, 2, 3))
                e += w * (u[:, 0] ** 2 * v1[:, 0] + u[:, 1] ** 2 * v1[:, 1] + u[:, 2] ** 2 * v[:, 1]
                          + 2 * (u[:, 0] * u[:, 1] * v2[:, 0] + u[:, 0] * u[:, 2] * v2[:, 1]
                                 + u[:, 1] * u[:, 2] * v3[:, 0]))
        return d, e

    npix = t["npix"].cpu().numpy()
    for q0, q1, ns in _groups(npix, _pow2_up, 1 << 23):
        j = torch.arange(ns, device=DEV)
        keep = j[None, :] < t["npix"][q0:q1, None]
        row, col = keep.nonzero(as_tuple=True)
        q = row + q0
        at = t["off"][q] + col
        u = t["step"][q0:q1].double()
        u = (u / u.norm(dim=1, keepdim=True))[row] if case["interp"] == "wide" else None
        d, e = interpolate(t["origin"][q] + col[:, None] * t["step"][q], u)
        if ns >= 2:
            d = d + _delta_s(_normals_ds(st["seed"], q0, q1, ns), ns, PS_AMP, PS_KCUT)[row, col]
        out["dens"][at], out["eta"][at] = d, e
        if case["fgpa"]:
            chi = t["chi0"][q] - col.double() * DPIX
            x = 1.0 + _z_of_chi(chi)
            a, b, c = (p[0] + x * (p[1] + x * p[2]) for p in co)
            flux = torch.exp(-a * torch.exp(b * (d + c * e)))
            out["flux"][at] = flux
            if case["bins"]:
                fsum += _bin_sums(chi, flux, edges)
    if case["bins"]:
        out["fsum"], out["count"] = fsum, None
    return out


def _bin_sums(chi, flux, edges):
    b = torch.searchsorted(edges, chi, right=True) - 1
    ok = (b >= 0) & (b < edges.numel() - 1)
    return torch.zeros(edges.numel() - 1, dtype=torch.float64, device=DEV).index_add_(0, b[ok], flux[ok])


def _modes_bins(n_p, dv, device=DEV):
    """k bin of modes 1..n_p/2 (-1: none)."""
    k = 2 * math.pi * torch.arange(1, n_p // 2 + 1, device=device, dtype=torch.float64) / (n_p * dv)
    e = torch.from_numpy(K_EDGES).to(device)
    b = torch.searchsorted(e, k, right=True) - 1
    return torch.where(b < len(K_EDGES) - 1, b, torch.full_like(b, -1))


def _n_p(v):
    return min(1 << (v.bit_length() - 1), 2048) if v >= 2 else 0


def _power_sums(rows, n_p, dv):
    """Sum over rows and modes of |X_m|^2 / n_p per k bin (32)."""
    p = torch.fft.rfft(rows, dim=1)[:, 1:].abs().square().sum(dim=0) / n_p
    b = _modes_bins(n_p, dv)
    ok = b >= 0
    return torch.zeros(32, dtype=torch.float64, device=DEV).index_add_(0, b[ok], p[ok])


def _mode_counts(npix, dv):
    """Modes per k bin over all skewers."""
    cnt = torch.zeros(32, dtype=torch.float64, device=DEV)
    for n_p, c in zip(*np.unique([_n_p(int(v)) for v in npix], return_counts=True)):
        if n_p:
            b = _modes_bins(int(n_p), dv)
            cnt += float(c) * torch.bincount(b[b >= 0], minlength=32).double()
    return cnt


def _exact_post(case, seed):
    st = prepare(case, seed)
    t = st["t"]
    npix = t["npix"].cpu().numpy()
    flux = torch.zeros(t["total"], dtype=torch.float64, device=DEV)
    fsum = torch.zeros(len(Z_EDGES) - 1, dtype=torch.float64, device=DEV)
    count = torch.zeros_like(fsum)
    table = (st["ps_k"], st["ratio"].double())
    for q0, q1, ns in _groups(npix, _pow2_up, 1 << 24):
        j = torch.arange(ns, device=DEV)
        row, col = (j[None, :] < t["npix"][q0:q1, None]).nonzero(as_tuple=True)
        q = row + q0
        at = t["off"][q] + col
        d = st["dens"][at].double()
        if case["delta_s"] and ns >= 2:
            d = d + _delta_s(_normals_ds(st["seed"], q0, q1, ns), ns, PS_AMP, PS_KCUT, table)[row, col]
        chi = t["chi0"][q] - col.double() * DPIX
        x = 1.0 + _z_of_chi(chi)
        a, b, c = (p[0] + x * (p[1] + x * p[2]) for p in FGPA)
        f = torch.exp(-a * torch.exp(b * (d + c * st["eta"][at].double())))
        flux[at] = f
        fsum += _bin_sums(chi, f, st["edges"])
        count += _bin_sums(chi, torch.ones_like(f), st["edges"])
    fbar = torch.where(count > 0, fsum / count.clamp(min=1), 1.0)
    dv = DPIX * _km_s(2.5)
    psum = torch.zeros(32, dtype=torch.float64, device=DEV)
    for q0, q1, n_p in _groups(npix, _n_p, 1 << 24):
        if n_p < 2:
            continue
        j = torch.arange(n_p, device=DEV)
        chi = t["chi0"][q0:q1, None] - j.double() * DPIX
        b = (torch.searchsorted(st["edges"], chi, right=True) - 1).clamp(0, fbar.numel() - 1)
        rows = flux[t["off"][q0:q1, None] + j] / fbar[b] - 1.0
        psum += dv * _power_sums(rows, n_p, dv)
    return dict(flux=flux, fsum=fsum, count=None, psum=psum, pcount=None)


def _exact_labels(case, seed):
    st = prepare(case, seed)
    t, k = st["t"], case["draws"]
    npix = t["npix"].cpu().numpy()
    if case["delta_s"] and t["total"] * k > 1 << 28:
        return None
    dens, eta = st["dens"].double(), st["eta"].double()
    zz = {}
    y = torch.zeros((k, 33), dtype=torch.float64, device=DEV)
    for i, dr in enumerate(st["draws"]):
        a, b, c, z = dr if not case["delta_s"] else (dr[0], dr[1], 1.2, 2.5)
        d = dens
        if case["delta_s"]:
            d = dens.clone()
            for q0, q1, ns in _groups(npix, _pow2_up, 1 << 23):
                if ns < 2:
                    continue
                if (q0, ns) not in zz:
                    zz[(q0, ns)] = _normals_ds(st["seed"], q0, q1, ns)
                ds = _delta_s(zz[(q0, ns)], ns, dr[2], dr[3])
                j = torch.arange(ns, device=DEV)
                row, col = (j[None, :] < t["npix"][q0:q1, None]).nonzero(as_tuple=True)
                d[t["off"][row + q0] + col] += ds[row, col]
        f = torch.exp(-a * torch.exp(b * (d + c * eta)))
        fbar = f.mean()
        dv = DPIX * _km_s(z)
        p = torch.zeros(32, dtype=torch.float64, device=DEV)
        for q0, q1, n_p in _groups(npix, _n_p, 1 << 25):
            if n_p >= 2:
                rows = f[t["off"][q0:q1, None] + torch.arange(n_p, device=DEV)]
                p += _power_sums(rows, n_p, dv)
        y[i, 0] = fbar
        y[i, 1:] = dv * p / (fbar * fbar * _mode_counts(npix, dv))
    return y


def _exact_train(case, seed):
    st = prepare(case, seed)
    p = st["params"].double().clone().requires_grad_(True)
    h = st["x0"].double()
    for i, (w, b, fan) in enumerate(_layers(case["n_out"])):
        h = h @ p[w[0]:w[1]].view(fan, -1) + p[b[0]:b[1]]
        if i < 3:
            h = torch.nn.functional.gelu(h)
    loss = (h - st["tgt"].double()).square().mean()
    grad, = torch.autograd.grad(loss, p)
    return dict(grad=grad, loss=loss.detach().reshape(1))


def _exact_quasars(case, seed):
    st = prepare(case, seed)
    out = []
    for f in st["fields"]:
        v = L.box_view(f, case["n"])
        for c in (0, 1):
            x = v[..., c].double()
            m = x.mean()
            out += [m, x.square().mean() - m * m]
            del x
    return dict(moments=torch.stack(out), count=None, pos=None)


def _growth(z):
    x, w = np.polynomial.legendre.leggauss(200)

    def d(a):
        t = 0.5 * math.sqrt(a) * (x + 1.0)
        ae2 = OMEGA_M / t ** 2 + (1 - OMEGA_M) * t ** 4
        return math.sqrt(OMEGA_M / a ** 3 + 1 - OMEGA_M) * 0.5 * math.sqrt(a) * np.sum(w * 2 * t / ae2 ** 1.5)
    return d(1.0 / (1.0 + z)) / d(1.0)


def _exact_lognormal(case, seed):
    st = prepare(case, seed)
    s, rmax, n_r = case["smooth"], case["rmax"], case["n_r"]
    kmax = 12.0 / s
    m = int(2 * math.ceil(kmax / (2 * min(0.1 / rmax, kmax / 64.0))))
    h = kmax / m
    k = h * np.arange(1, m + 1)
    w = np.where(np.arange(1, m + 1) % 2 == 1, 4.0, 2.0)
    w[-1] = 1.0
    f = w * h / 3.0 * _pk_amp(st["sigma8"]) * _pk_shape(k) * np.exp(-(k * s) ** 2) * k
    f, k = torch.from_numpy(f).to(DEV), torch.from_numpy(k).to(DEV)
    dr = rmax / (n_r - 1)
    r = dr * torch.arange(n_r, dtype=torch.float64, device=DEV)
    xi = torch.empty_like(r)
    step = max(1, (1 << 27) // m)
    for i in range(0, n_r, step):
        rr = r[i:i + step]
        xi[i:i + step] = (torch.sin(rr[:, None] * k) @ f) / rr.clamp(min=1e-300)
    xi[0] = (f * k).sum()
    xi = xi / (2 * math.pi ** 2)
    b0 = 3.7 * ((1 + QSO_Z[0]) / 3.33) ** 1.7 * _growth(QSO_Z[1]) * (1 + QSO_Z[1]) / (1 + QSO_Z[0])
    i = torch.arange(n_r, device=DEV)
    wr = torch.where((i == 0) | (i == n_r - 1), 1.0, torch.where(i % 2 == 1, 4.0, 2.0).double())
    g = wr * dr / 3.0 * torch.log1p(b0 * b0 * xi) * r
    kv = st["k"]
    pq = 4 * math.pi * (torch.sin(kv[:, None] * r) @ g) / kv
    return dict(pq=torch.maximum(pq, 1e-12 * pq.max()), xi=xi)


def exact(case, seed):
    fn = dict(box=lambda: _exact_box(case, int(seed) * 2 + 1), skewers=lambda: _exact_skewers(case, seed),
              post=lambda: _exact_post(case, seed), labels=lambda: _exact_labels(case, seed),
              train=lambda: _exact_train(case, seed), quasars=lambda: _exact_quasars(case, seed),
              lognormal=lambda: _exact_lognormal(case, seed))[case["kind"]]
    return fn()
