"""The performance cases of this framework: finite-temperature Lanczos work as its users call it.

A program that uses the framework builds a cluster graph and an S^z sector
once, keeps them (with a workspace or a plan), and then calls

  hv        y = H x for one vector or a block of vectors (`ftlm.hv`), or one
            device's share of the rows (`ftlm.hv_rows`);
  lanczos   R Lanczos chains of M steps in one sector (`ftlm.lanczos`);
  request   one FTLM estimate: chains, host Ritz values and the thermal
            reduction (`driver.sector_samples`, `ftlm.thermo`);
  plan      the chains of every S^z >= 0 sector of a lattice (`Plan.run`).

Every size comes from the repository's tests, benchmark and request stream:
rings of 12 to 34 sites, the 6 x 4 J1-J2 lattice, the icosidodecahedron, the
random clusters of the request stream, and the icosahedron at higher spin.
No case holds a vector block of 2^31 entries or more: torch's own indexing is
not to be relied on above that, and the outputs are read with it.
"""
import math

import numpy as np
import torch

from ftlm_inputs import graphs
from paper_2605_26261_amd import driver, ftlm

DEV = "cuda"
MODES = {"cr": ftlm.CR, "clt": ftlm.CLT, "lin": ftlm.LIN, "full": ftlm.FULL}
TORCH_DTYPE = {"f32": torch.float32, "f64": torch.float64}
DTYPE = {"f32": ftlm.F32, "f64": ftlm.F64}
DIST = {"pm1": ftlm.PM1, "gauss": ftlm.GAUSS}


def listed():
    return [
        # The smallest whole call: the 12-site ring of the exact-diagonalisation
        # checks, 924 states, in FP64. Nothing but latency and launches.
        {"name": "lanczos_ring12_f64", "do": "lanczos", "graph": "ring", "sites": 12, "n_up": 6, "mode": "cr",
         "dtype": "f64", "cols": 8, "steps": 40, "dist": "pm1"},
        # A single product on a small sector (48,620 states), the inner call of
        # a user's own Krylov loop: a launch with little under it.
        {"name": "hv_ring18_f32x1", "do": "hv", "graph": "j1j2_ring", "sites": 18, "n_up": 9, "mode": "cr",
         "dtype": "f32", "cols": 1},
        # One request of the exchange-fit stream at an odd site count: a random
        # cluster, M = 1/2 (352,716 states), R = 16, 80 steps, then Ritz values and
        # thermodynamics.
        {"name": "request_cluster21", "do": "request", "graph": "cluster", "sites": 21, "n_up": 11, "mode": "cr",
         "dtype": "f32", "cols": 16, "steps": 80, "dist": "pm1"},
        # The precision study's chains at spin 1: icosahedron, 73,789 states, FP64.
        {"name": "lanczos_ico12_s1_f64", "do": "lanczos", "graph": "icosahedron", "sites": 12, "two_s": 2, "n_up": 12,
         "mode": "cr", "dtype": "f64", "cols": 8, "steps": 60, "dist": "gauss"},
        # A block product on a mid-sized lattice sector (2.7 million states) through
        # the compressed lookup table.
        {"name": "hv_square24_clt_f32x8", "do": "hv", "graph": "square", "sites": 24, "n_up": 12, "mode": "clt",
         "dtype": "f32", "cols": 8},
        # The whole lattice: 13 sectors of 1 to 2.7 million states in one plan.
        {"name": "plan_square24", "do": "plan", "graph": "square", "sites": 24, "mode": "cr", "dtype": "f32",
         "cols": 32, "steps": 24, "dist": "pm1"},
        # One vector of the headline sector (155,117,520 states), without tables.
        {"name": "hv_icosidod30_f32x1", "do": "hv", "graph": "icosidodecahedron", "sites": 30, "n_up": 15, "mode": "cr",
         "dtype": "f32", "cols": 1},
        # Double precision through the compressed table, two vectors.
        {"name": "hv_icosidod30_clt_f64x2", "do": "hv", "graph": "icosidodecahedron", "sites": 30, "n_up": 15,
         "mode": "clt", "dtype": "f64", "cols": 2},
        # The block product of the headline sector at its best width per vector.
        {"name": "hv_icosidod30_f32x8", "do": "hv", "graph": "icosidodecahedron", "sites": 30, "n_up": 15, "mode": "cr",
         "dtype": "f32", "cols": 8},
        # One batch of the headline run's Gaussian chains at the batch width that
        # the autotuner picks, cut to 16 steps.
        {"name": "lanczos_icosidod30", "do": "lanczos", "graph": "icosidodecahedron", "sites": 30, "n_up": 15,
         "mode": "cr", "dtype": "f32", "cols": 8, "steps": 16, "dist": "gauss"},
        # More than 32 sites: 64-bit labels (286,097,760 states), four vectors.
        {"name": "hv_ring34_f32x4", "do": "hv", "graph": "j1j2_ring", "sites": 34, "n_up": 11, "mode": "cr",
         "dtype": "f32", "cols": 4},
        # Spin 5/2 icosahedron, M = 0 (144,840,476 states), one vector.
        {"name": "hv_ico12_s52_f32x1", "do": "hv", "graph": "icosahedron", "sites": 12, "two_s": 5, "n_up": 30,
         "mode": "cr", "dtype": "f32", "cols": 1},
    ]


# ---- sizes --------------------------------------------------------------------------

def bonds_of(case, seed):
    """The bond list [(i, j, J)] of the case; the random clusters are drawn from the seed."""
    g, n = case["graph"], case["sites"]
    if g == "ring":
        return graphs.ring(n)
    if g == "j1j2_ring":
        return graphs.j1j2_ring(n)
    if g == "square":
        return graphs.square_j1j2(n // 4, 4)
    if g == "icosidodecahedron":
        return graphs.icosidodecahedron()
    if g == "dodecahedron":
        return graphs.dodecahedron()
    if g == "icosahedron":
        return graphs.icosahedron()
    return graphs.random_cluster(n, np.random.default_rng(seed))


def bond_count(case):
    n = case["sites"]
    return {"ring": n, "j1j2_ring": 2 * n, "square": 4 * n, "icosidodecahedron": 60, "dodecahedron": 30,
            "icosahedron": 30, "cluster": round(1.75 * n)}[case["graph"]]


def dimension(n, two_s, a):
    """Eq. 15: digit strings of n digits 0..two_s with sum a."""
    d = [1]
    for _ in range(n):
        d = [sum(d[q] for q in range(max(0, s - two_s), min(len(d) - 1, s) + 1)) for s in range(len(d) + two_s)]
    return d[a] if 0 <= a < len(d) else 0


def plan_sectors(case):
    return list(range((case["sites"] + 1) // 2, case["sites"] + 1))


def states(case):
    if case["do"] == "plan":
        return sum(dimension(case["sites"], 1, a) for a in plan_sectors(case))
    return dimension(case["sites"], case.get("two_s", 1), case["n_up"])


def draw(rng):
    """One more case of the same kinds and ranges."""
    for _ in range(1000):
        c = _draw(rng)
        d = states(c)
        if d < 200:
            continue
        es = 8 if c["dtype"] == "f64" else 4
        cells = d * c["cols"]
        if cells >= 1 << 31 or cells * es * (1 if c["do"] == "hv" else 2) > 26e9:
            continue
        # held under the largest listed case's time: a block of fewer than four columns
        # costs about as much as one of four, a bond of higher spin has two terms
        cost = d * max(4, c["cols"]) * es / 4 * bond_count(c) * c.get("steps", 1)
        if cost <= 1.1e12 * (0.5 if c.get("two_s", 1) > 1 else 1.0):
            return c
    raise RuntimeError("no case drawn")


def _draw(rng):
    do = rng.choice(["hv", "hv", "hv", "hv_spin", "lanczos", "lanczos", "request", "plan"])
    if do == "plan":
        n = rng.choice([12, 16, 20, 24])
        return {"do": "plan", "graph": rng.choice(["square", "j1j2_ring", "cluster"]) if n > 12 else "ring", "sites": n,
                "mode": rng.choice(["cr", "cr", "clt"]), "dtype": rng.choice(["f32", "f32", "f64"]),
                "cols": rng.choice([4, 7, 8, 16, 32]), "steps": rng.randint(10, 30), "dist": rng.choice(["pm1", "gauss"])}
    if do == "request":
        n = rng.randint(16, 28)
        return {"do": "request", "graph": "cluster", "sites": n, "n_up": (n + 1) // 2 + rng.randint(0, n // 4),
                "mode": rng.choice(["cr", "cr", "clt"]), "dtype": "f32", "cols": 16, "steps": rng.randint(40, 80),
                "dist": "pm1"}
    spin = do == "hv_spin" or (do == "lanczos" and rng.random() < 0.25)
    if spin:
        two_s = rng.choice([2, 3, 4, 5])
        c = {"graph": "icosahedron", "sites": 12, "two_s": two_s, "n_up": 6 * two_s + rng.randint(0, 4 * two_s),
             "mode": rng.choice(["cr", "clt"])}
    else:
        n = rng.randint(12, 34)
        g = rng.choice(["j1j2_ring", "cluster", "cluster", "ring"])
        if n in (20, 24, 28) and rng.random() < 0.4:
            g = "square"
        if n == 30 and rng.random() < 0.7:
            g = "icosidodecahedron"
        if n == 20 and rng.random() < 0.3:
            g = "dodecahedron"
        n_up = (n + 1) // 2 + rng.randint(0, n // 5)
        if n >= 33:
            n_up = rng.randint(8, 11)
        c = {"graph": g, "sites": n, "n_up": n_up,
             "mode": "cr" if n > 30 else rng.choice(["cr", "cr", "cr", "clt", "clt", "lin", "full"])}
    if do.startswith("hv"):
        c = {"do": "hv", **c, "dtype": rng.choice(["f32", "f32", "f32", "f64"]),
             "cols": rng.choice([1, 1, 1, 2, 3, 4, 5, 6, 8, 8, 10, 12, 16, 20, 32])}
        if rng.random() < 0.15:
            c["share"] = rng.choice([2, 4, 8])
        return c
    return {"do": "lanczos", **c, "dtype": rng.choice(["f32", "f32", "f64"]),
            "cols": rng.choice([1, 2, 4, 5, 8, 8, 10, 12, 16, 20]), "steps": rng.randint(6, 60),
            "dist": rng.choice(["pm1", "gauss"])}


# ---- what a program holds, and one pass ------------------------------------------------

def prepare(case, seed):
    bonds = bonds_of(case, seed)
    s = {"case": case, "bonds": bonds, "seed": int(seed), "graph": ftlm.Graph(case["sites"], bonds)}
    mode = MODES[case["mode"]]
    if case["do"] == "plan":
        s["plan"] = ftlm.Plan(s["graph"], plan_sectors(case), mode, case["cols"], case["steps"], DTYPE[case["dtype"]])
        return s
    s["sector"] = ftlm.Sector(case["sites"], case["n_up"], mode, two_s=case.get("two_s", 1))
    if case["do"] == "hv":
        s["x"] = start_block(case, seed)
        s["rows"] = share_rows(case)
        rows = s["rows"][1]
        s["y"] = torch.empty((rows,) + tuple(s["x"].shape[1:]), dtype=s["x"].dtype, device=DEV)
    else:
        n = ftlm.lanczos_workspace_bytes(s["sector"], case["cols"], DTYPE[case["dtype"]])
        s["work"] = torch.empty(n, dtype=torch.uint8, device=DEV)
        s["temps"] = driver.log_temperatures()
    return s


def start_block(case, seed):
    """The vectors of a Krylov iteration: independent Gaussian components."""
    gen = torch.Generator(device=DEV).manual_seed(int(seed))
    d, b = states(case), case["cols"]
    return torch.randn((d,) if b == 1 else (d, b), dtype=TORCH_DTYPE[case["dtype"]], device=DEV, generator=gen)


def share_rows(case):
    """(first row, rows) of the product: all of them, or the second of `share` row shares."""
    d, k = states(case), case.get("share", 1)
    return (0, d) if k == 1 else (d // k, d // k)


def run(state):
    c = state["case"]
    if c["do"] == "hv":
        if "share" in c:
            ftlm.hv_rows(state["sector"], state["graph"], state["x"], state["y"], *state["rows"])
        else:
            ftlm.hv(state["sector"], state["graph"], state["x"], state["y"])
        return {"y": state["y"]}
    if c["do"] == "lanczos":
        a, b, k = ftlm.lanczos(state["sector"], state["graph"], state["seed"], 0, c["cols"], c["steps"], DIST[c["dist"]],
                               DTYPE[c["dtype"]], work=state["work"])
        return {"alpha": a, "beta": b, "steps": k}
    if c["do"] == "plan":
        a, b, k = state["plan"].run(state["seed"], DIST[c["dist"]])
        return {"alpha": a, "beta": b, "steps": k}
    rec = driver.sector_samples(state["sector"], state["graph"], c["cols"], c["steps"], state["seed"], DIST[c["dist"]],
                                DTYPE[c["dtype"]], work=state["work"])
    out = ftlm.thermo(c["sites"], [rec], state["temps"])
    return {"alpha": rec["alpha"], "beta": rec["beta"], "steps": rec["steps"], "E": out["E"], "C": out["C"],
            "lnZ": out["lnZ"]}


def work(case):
    """hv: x read once, y written once. A Lanczos step reads u_k and u_{k-1}
    and writes w, and its second half (alpha is a sum over all of w) reads u_k
    and w and writes u_{k+1}; the start block is written once. A flip term is
    one multiply-add per vector, about half of the bonds flip."""
    d, b = states(case), case["cols"]
    es = 8 if case["dtype"] == "f64" else 4
    nb = bond_count(case) * (2 if case.get("two_s", 1) > 1 else 1)
    if case["do"] == "hv":
        rows = share_rows(case)[1]
        return {"bytes": (d + rows) * b * es, "flops": rows * b * (nb + 2)}
    m = case["steps"]
    return {"bytes": d * b * es * (6 * m + 1), "flops": d * b * m * (nb + 10)}


# ---- the same numbers in 64 bits, in plain torch -----------------------------------------

class Exact:
    """H x (Eq. 12) in FP64 over base-(two_s + 1) labels in ascending order.
    A label splits into a high and a low part; the sector's index of a label is
    the number of sector labels with a smaller high part plus the rank of the
    low part among the low parts of its digit sum."""

    def __init__(self, case, seed):
        self.n, self.two_s, self.a = case["sites"], case.get("two_s", 1), case["n_up"]
        self.d, self.bonds = self.two_s + 1, bonds_of(case, seed)
        self.low = self.n // 2
        n_lo, n_hi = self.d ** self.low, self.d ** (self.n - self.low)
        s_lo, s_hi = self.sums(n_lo), self.sums(n_hi)
        order = torch.argsort(s_lo, stable=True)
        count = torch.bincount(s_lo, minlength=self.n * self.two_s + 1)
        first = torch.cumsum(count, 0) - count
        self.rank_lo = torch.empty(n_lo, dtype=torch.int64, device=DEV)
        self.rank_lo[order] = torch.arange(n_lo, device=DEV) - first[s_lo[order]]
        need = self.a - s_hi
        per = torch.where(need >= 0, count[need.clamp(0)], torch.zeros_like(need))
        self.base = torch.cumsum(per, 0) - per
        self.dim = int(per.sum())
        high = torch.repeat_interleave(torch.arange(n_hi, device=DEV, dtype=torch.int32), per).to(torch.int64)
        j = torch.arange(self.dim, device=DEV) - self.base[high]
        j += first[need.clamp(0)][high]
        self.label = order[j] + high * n_lo
        self.n_lo = n_lo

    def sums(self, count):
        x = torch.arange(count, device=DEV)
        s = torch.zeros_like(x)
        while count > 1:
            s += x % self.d
            x = x // self.d
            count //= self.d
        return s

    def index(self, label):
        return self.base[label // self.n_lo] + self.rank_lo[label % self.n_lo]

    def hv(self, x, row0=0, rows=None):
        """Rows [row0, row0 + rows) of H x for x of [dim, B] in FP64."""
        rows = self.dim if rows is None else rows
        out = torch.empty((rows, x.shape[1]), dtype=torch.float64, device=DEV)
        s = 0.5 * self.two_s
        for r in range(0, rows, 1 << 24):
            e = min(rows, r + (1 << 24))
            lab = self.label[row0 + r:row0 + e]
            diag = torch.zeros(e - r, dtype=torch.float64, device=DEV)
            acc = torch.zeros((e - r, x.shape[1]), dtype=torch.float64, device=DEV)
            for i, j, J in self.bonds:
                pi, pj = self.d ** i, self.d ** j
                ai, aj = lab // pi % self.d, lab // pj % self.d
                mi, mj = ai - s, aj - s
                diag += J * mi * mj
                for step, on, f in (
                        (pi - pj, (ai < self.two_s) & (aj > 0), (s * (s + 1) - mi * (mi + 1)) * (s * (s + 1) - mj * (mj - 1))),
                        (pj - pi, (ai > 0) & (aj < self.two_s), (s * (s + 1) - mi * (mi - 1)) * (s * (s + 1) - mj * (mj + 1)))):
                    at = on.nonzero()[:, 0]
                    acc.index_add_(0, at, 0.5 * J * f[at].sqrt()[:, None] * x[self.index(lab[at] + step)])
            out[r:e] = acc + diag[:, None] * x[row0 + r:row0 + e]
        return out


_M64 = (1 << 64) - 1


def _mix(z):
    z = ((z ^ (z >> 30)) * 0xbf58476d1ce4e5b9) & _M64
    z = ((z ^ (z >> 27)) * 0x94d049bb133111eb) & _M64
    return z ^ (z >> 31)


def _signed(v):
    v &= _M64
    return v - (1 << 64) if v >> 63 else v


def _mix_t(z):
    """SplitMix64's output function on int64 tensors (logical shifts)."""
    def shr(v, k):
        return (v >> k) & ((1 << (64 - k)) - 1)
    z = (z ^ shr(z, 30)) * _signed(0xbf58476d1ce4e5b9)
    z = (z ^ shr(z, 27)) * _signed(0x94d049bb133111eb)
    return z ^ shr(z, 31)


def exact_starts(case, seed, dim):
    """The normalised start vectors: SplitMix64 streams keyed by (seed, sector, sample)."""
    gamma = 0x9e3779b97f4a7c15
    i = torch.arange(dim, device=DEV)
    cols = []
    for r in range(case["cols"]):
        key = _mix((int(seed) + gamma) & _M64)
        for word in (case["n_up"], r):
            key = _mix(((key ^ word) + gamma) & _M64)
        if case["dist"] == "pm1":
            v = torch.where(_mix_t((i + 1) * _signed(gamma) + _signed(key)) < 0, -1.0, 1.0).double()
        else:
            u, w = (_mix_t((2 * i + k) * _signed(gamma) + _signed(key)) for k in (1, 2))
            u = (((u >> 11) & ((1 << 53) - 1)) + 1).double() * 2.0 ** -53
            w = ((w >> 11) & ((1 << 53) - 1)).double() * 2.0 ** -53
            v = torch.sqrt(-2.0 * torch.log(u)) * torch.cos(2.0 * math.pi * w)
        cols.append(v / v.norm())
    return torch.stack(cols, dim=1)


def exact(case, seed):
    """hv: the product in 64 bits. Chains: alpha and beta of the first steps
    are comparable between precisions, later ones are not (rounding decides
    them once Ritz values converge), so only short runs have a value."""
    rows = states(case)
    if case["do"] == "hv":
        if rows * case["cols"] * bond_count(case) * (3 if case.get("two_s", 1) > 1 else 1) > 8e10:
            return None
        e = Exact(case, seed)
        x = start_block(case, seed).double()
        x = x[:, None] if x.dim() == 1 else x
        y = e.hv(x, *share_rows(case))
        return {"y": y[:, 0] if case["cols"] == 1 else y}
    if case["do"] != "lanczos" or case["steps"] > 12:
        return None
    if rows * case["cols"] * bond_count(case) * case["steps"] > 5e10 or rows < 1000:
        return None
    e = Exact(case, seed)
    q, prev = exact_starts(case, seed, e.dim), None
    a, b = [], []
    for _ in range(case["steps"]):
        w = e.hv(q)
        if prev is not None:
            w -= b[-1] * prev
        a.append((q * w).sum(0))
        w -= a[-1] * q
        b.append(w.norm(dim=0))
        prev, q = q, w / b[-1]
    return {"alpha": torch.stack(a, 1), "beta": torch.stack(b, 1), "steps": None}
