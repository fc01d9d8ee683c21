"""The work that a user of octfd has it do, through the public entry points of the Python binding.

A case names a call, a kind of right-hand side and a tree.  Trees follow the recipes of synthdata: octants of level
lmin refined up to lmax around two seed points, `radius` (a length in the unit cube) at level lmin and `ratio` times
the last one at each further level; "rand" seeds lie anywhere in the middle of the cube, "orbit" seeds opposite each
other on a circle.  The tree belongs to the case; the fields on it are made from the seed.

Calls:
  rhs       rhs_eval_zipped: one right-hand side, zipped in and out (diagnostics, other integrators)
  step      rk_step: one Runge-Kutta step with the clamped ghost rule
  static    rk_step_static: the same in the library's own workspace (callers that cannot allocate)
  centred   rk_step_centred: one step with the centred ghost rule, the one for long evolutions
  pipeline  unzip, rhs_eval, zip: a caller that works on padded blocks between the calls
  regrid    the tree after the seeds have moved, its transfer plan, its tables on the GPU, all fields carried over
"""
import math

import numpy as np
import torch

import paper_2007_12792_amd as octfd
import synthdata as sd

BLOCK = 512
PADDED = 14 ** 3


def listed():
    return [
        # first look at a uniform grid, or a unit of work in a loop of many small ones: one launch
        case("derivs_uniform_512", "rhs", "DERIVS", 3, 3),
        # derivatives of one field on an ordinary adaptive tree
        case("derivs_9213", "rhs", "DERIVS", 3, 6, radius=0.12),
        # small runs, where a step is a chain of short launches: a coarse exploratory run of the wave system with the
        # rule for evolutions, and a caller without a workspace
        case("wave_centred_834", "centred", "WAVE", 3, 5, radius=0.0573, ratio=0.667),
        case("burgers_static_834", "static", "BURGERS", 3, 5, radius=0.0573, ratio=0.667),
        # production runs of the two small systems
        case("wave_centred_47783", "centred", "WAVE", 3, 7, radius=0.12),
        case("burgers_step_47783", "step", "BURGERS", 3, 7, radius=0.12),
        # analysis on padded blocks: the three calls one by one
        case("wave_pipeline_47783", "pipeline", "WAVE", 3, 7, radius=0.12),
        case("syn24_pipeline_21064", "pipeline", "SYN24", 3, 7, radius=0.085),
        # the 24-field system: smallest, one evaluation on an ordinary tree, a step of the benchmark's tree
        case("syn24_step_792", "step", "SYN24", 3, 5, style="orbit", radius=0.0668, ratio=0.643),
        case("syn24_rhs_21064", "rhs", "SYN24", 3, 7, radius=0.085),
        case("syn24_step_102075", "step", "SYN24", 3, 9, style="orbit", radius=0.1, ratio=0.83),
        # the regrid between two stretches of steps: host tables and one pass over all fields
        case("syn24_regrid_27791", "regrid", "SYN24", 3, 8, style="orbit", radius=0.1, ratio=0.83, phase=0.026),
    ]


def case(name, call, kind, lmin, lmax, style="rand", radius=0.0, ratio=1.0, tree_seed=1, phase=0.0):
    c = dict(call=call, kind=kind, lmin=lmin, lmax=lmax, style=style, radius=radius, ratio=ratio, tree_seed=tree_seed, phase=phase)
    return dict(c, name=name) if name else c


#: (call, kind, most blocks): what draw() takes from.  The bound keeps a drawn case under the largest listed one.
DRAWN = [("rhs", "DERIVS", 100000), ("rhs", "WAVE", 100000), ("rhs", "BURGERS", 100000), ("rhs", "SYN24", 60000),
         ("step", "WAVE", 100000), ("step", "BURGERS", 100000), ("step", "SYN24", 60000), ("static", "WAVE", 4500),
         ("centred", "WAVE", 100000), ("centred", "BURGERS", 100000), ("centred", "SYN24", 60000),
         ("pipeline", "DERIVS", 60000), ("pipeline", "WAVE", 60000), ("pipeline", "SYN24", 20000),
         ("regrid", "WAVE", 40000), ("regrid", "SYN24", 40000)]


def draw(rng):
    call, kind, most = rng.choice(DRAWN)
    want = math.exp(rng.uniform(math.log(519), math.log(0.9 * most)))
    style = "orbit" if call == "regrid" else rng.choice(("rand", "orbit"))
    lmin = rng.choice((3, 4)) if want > 6000 else 3
    lmax = rng.randint(lmin + 1, min(9, lmin + 1 + int(math.log2(want / 400))))
    ratio = round(rng.uniform(0.6, 1.0), 3)
    c = case("", call, kind, lmin, lmax, style, 0.0, ratio, rng.randrange(1 << 20))
    # the radius that brings the number of blocks near the one wanted, by halving
    lo, hi = 0.001, 0.5
    for _ in range(9):
        c["radius"] = round(math.sqrt(lo * hi), 5)
        n = most if rough_size(c) > 4 * most else tree(c).n
        lo, hi = (c["radius"], hi) if n < want else (lo, c["radius"])
    c["radius"] = round(lo, 5)
    if call == "regrid":     # the seeds move by about one block of the finest level: no leaf changes by two levels
        c["phase"] = round(rng.uniform(0.3, 1.0) * 2.0 ** -lmax / 0.15, 5)
        while not can_regrid(c):
            c["phase"] /= 2
    return c


def rough_size(c):
    """Blocks inside the balls around the two seeds, level by level: enough to keep draw() from building huge trees."""
    return sum(8.0 ** (c["lmin"] + k + 1) * min(1.0, 8.4 * (c["radius"] * c["ratio"] ** k) ** 3) for k in range(c["lmax"] - c["lmin"]))


def tree_recipe(c, phase=0.0):
    radii = [int(c["radius"] * c["ratio"] ** k * sd.Q) for k in range(c["lmax"] - c["lmin"])]
    return c["lmin"], c["lmax"], sd.seed_points(c["style"], c["tree_seed"], phase), np.asarray(radii, dtype=np.uint32)


def tree(c, phase=0.0):
    return octfd.Tree.build(*tree_recipe(c, phase))


def can_regrid(c):
    try:
        octfd.Transfer(tree(c), tree(c, c["phase"]))
        return True
    except octfd.OctfdError:
        return False


#: the workloads of synthdata whose fields a kind starts from
FIELDS = {"DERIVS": "C2", "WAVE": "C3", "BURGERS": "C3B", "SYN24": "C4"}


def fields(c, leaves, seed):
    """The kind's initial fields; those that synthdata makes without noise get other amplitudes with another seed."""
    u = sd.make_fields(FIELDS[c["kind"]], leaves, seed % (1 << 40), device="cuda")
    if c["kind"] in ("WAVE", "BURGERS"):
        u += 1e-3 * sd.normal_noise(seed % (1 << 40) + 101, u.numel(), "cuda").view(u.shape)
    return u


def time_step(c):
    """A step that a long run could take: passes may be many, and the state has to stay a solution through all of them."""
    h = 2.0 ** -(c["lmax"] + 3)
    return h * h / 1024 if c["kind"] == "SYN24" else h / 1024    # the 24-field system is parabolic


def empty(*shape):
    return torch.empty(shape, dtype=torch.float64, device="cuda")


def prepare(c, seed):
    kind = octfd.KINDS[c["kind"]]
    t = tree(c)
    t.upload()
    s = dict(call=c["call"], kind=kind, tree=t, u=fields(c, t.leaves, seed), sigma=0.0 if c["kind"] == "DERIVS" else sd.KO_SIGMA)
    if c["call"] in ("rhs", "pipeline"):
        s["out"] = empty(octfd.nvar_out(kind), t.n, 8, 8, 8)
    if c["call"] == "pipeline":
        s["padded"] = empty(octfd.nvar_in(kind), t.n, 14, 14, 14)
        s["rhs_padded"] = empty(octfd.nvar_out(kind), t.n, 14, 14, 14)
    if c["call"] in ("step", "static", "centred"):
        s["dt"] = time_step(c)
    if c["call"] == "step":
        s["workspace"] = empty(t.rk_workspace_bytes(kind) // 8)
    if c["call"] == "centred":
        s["workspace"] = empty(t.rk_centred_workspace_bytes(kind) // 8)
    if c["call"] == "regrid":
        s["moved"] = tree_recipe(c, c["phase"])
    return s


def run(s):
    t, kind, sigma = s["tree"], s["kind"], s["sigma"]
    if s["call"] == "rhs":
        t.rhs_eval_zipped(kind, s["u"], s["out"], sigma=sigma)
        return s["out"]
    if s["call"] == "step":
        t.rk_step(kind, s["u"], s["dt"], s["workspace"], sigma=sigma)
        return s["u"]
    if s["call"] == "static":
        t.rk_step_static(kind, s["u"], s["dt"], sigma=sigma)
        return s["u"]
    if s["call"] == "centred":
        t.rk_step_centred(kind, s["u"], s["dt"], s["workspace"], sigma=sigma)
        return s["u"]
    if s["call"] == "pipeline":
        t.unzip(s["u"], s["padded"])
        t.rhs_eval(kind, s["padded"], s["rhs_padded"], sigma=sigma)
        t.zip(s["rhs_padded"], s["out"])
        return s["padded"], s["out"]
    new = octfd.Tree.build(*s["moved"])
    plan = octfd.Transfer(t, new)
    new.upload()
    u = empty(s["u"].shape[0], new.n, 8, 8, 8)
    plan.apply(s["u"], u)
    return new.leaves, u


#: operations of one right-hand side at a point: a first derivative 9, a second 12, the sixth difference of an axis 8; the
#: mixed second derivatives of the 24-field system as one outer and 2.25 / 3 inner first derivatives each
RHS_FLOPS = {"DERIVS": 3 * 9 + 3 * 12 + 2, "WAVE": 3 * 12 + 2 + 2 * 28 + 2, "BURGERS": 9 + 28 + 2,
             "SYN24": 24 * (3 * 9 + 28 + 5 + 6 + 1 + 1 + 4) + 10 * (3 * 12 + 3 * 9 + 20 + 12) + 3 * 9}


def work(c):
    """Each call's inputs read once and its outputs written once."""
    kind = octfd.KINDS[c["kind"]]
    vi, vo = octfd.nvar_in(kind), octfd.nvar_out(kind)
    n = tree(c).n
    points = n * BLOCK
    if c["call"] == "regrid":
        to = tree(c, c["phase"]).n
        return {"bytes": 8 * vi * BLOCK * (n + to), "flops": 0}
    if c["call"] == "rhs":
        return {"bytes": 8 * (vi + vo) * points, "flops": RHS_FLOPS[c["kind"]] * points}
    if c["call"] == "pipeline":     # three calls: the padded arrays are outputs of one and inputs of the next
        return {"bytes": 8 * n * (vi * (BLOCK + 2 * PADDED) + 3 * vo * BLOCK), "flops": RHS_FLOPS[c["kind"]] * points}
    return {"bytes": 16 * vi * points, "flops": 4 * (RHS_FLOPS[c["kind"]] + 4 * vi) * points}


def tolerance(c):
    """Four times what the path differs by from itself with every sum unfused and in the compiler's order (measured on the
    listed trees).  A right-hand side divides by h and h squared, which magnifies the rounding of fields that are smooth on
    the grid; a step adds little to the state, and what is left is the rounding of the result."""
    if c["call"] in ("rhs", "pipeline"):
        return {"rel": 1e-10, "max": 4e-8} if c["kind"] == "SYN24" else {"rel": 1.2e-13, "max": 2.5e-11}
    return {"rel": 1e-15, "max": 2e-14}
