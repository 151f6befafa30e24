"""The calls this library's speed is judged on: what a program that relaxes fields with it does, through the
public entry points (the C ABI as the binding exposes it), from the smallest plates to the largest domains.

Two kinds of call:
  "solve"  a padded field comes in (jacobi_scatter), a schedule of iterations with residual norms runs
           (jacobi_run), the field goes out (jacobi_gather) - a whole job, so a repeated pass starts from the
           same field and gives the same result;
  "check"  no iterations: field in, halo exchange, residual norm, field out - what a program does that loads a
           state, makes its halos current for its own kernels, and reports how far from converged it is.
"""
import math

import torch

from paper_2210_01238_amd import harness

B = harness.B
NUMPY_NAME = {"f64": "float64", "f32": "float32"}
TORCH_TYPE = {"f64": torch.float64, "f32": torch.float32}


def _case(name, kind, dims, tiles, dtype="f64", iters=0, every=0, tblock=1):
    c = {"kind": kind, "dtype": dtype, "iters": iters, "every": every, "tblock": tblock}
    if name:
        c["name"] = name
    for i, (n, t) in enumerate(zip(dims, tiles)):
        c["n%d" % i] = n
        c["t%d" % i] = t
    return c


def _dims(case):
    return tuple(case["n%d" % i] for i in range(3) if "n%d" % i in case)


def _tiles(case):
    return tuple(case["t%d" % i] for i in range(3) if "t%d" % i in case)


def listed():
    return [
        # the smallest job: one small plate, 100 iterations; launches and synchronisation count, not bandwidth
        _case("plate_256", "solve", (256, 256), (1, 1), iters=100, every=100),
        # an ordinary plate, cut into tiles; both grids fit the caches many times over
        _case("plate_1024", "solve", (1024, 1024), (4, 4), iters=100, every=50),
        # fp32, tiles whose width fills neither a cache line nor a vector
        _case("ragged_2d_f32", "solve", (1500, 1110), (5, 3), "f32", iters=100, every=25),
        # two grids about the size of the last-level cache
        _case("square_4096", "solve", (4096, 4096), (4, 4), iters=100, every=100),
        # over-decomposed: 4096 small tiles
        _case("tiles_8192", "solve", (8192, 8192), (64, 64), iters=50, every=50),
        # the large 2-D domain, one exchange per iteration, a norm every 10
        _case("domain_16384", "solve", (16384, 16384), (8, 8), iters=20, every=10),
        # the same domain with several iterations per pass over memory
        _case("domain_16384_blocked", "solve", (16384, 16384), (8, 8), iters=50, every=10, tblock=12),
        # a small cube in eight blocks: the 3-D counterpart of the small plates
        _case("cube_64", "solve", (64, 64, 64), (2, 2, 2), iters=100, every=50),
        # fp32 blocks with odd extents
        _case("ragged_3d_f32", "solve", (210, 198, 250), (2, 2, 2), "f32", iters=40, every=20),
        # the 512^3 domain in 64 blocks
        _case("cube_512", "solve", (512, 512, 512), (4, 4, 4), iters=20, every=10),
        # the 1024 x 1024 x 768 domain in blocks of 128^3, several iterations per pass
        _case("paper_domain_blocked", "solve", (768, 1024, 1024), (6, 8, 8), iters=20, every=10, tblock=4),
        # state in, halos, norm, state out: no iterations
        _case("check_512_f32", "check", (512, 512, 512), (4, 4, 4), "f32"),
    ]


MOST_UPDATES = 5.0e9     # point updates of one call (the largest listed default-schedule call: 16384^2 x 20)


def draw(rng):
    """One more call of the same ranges."""
    three_d = rng.random() < 0.5
    kind = "check" if rng.random() < 0.15 else "solve"
    dtype = "f32" if rng.random() < 0.35 else "f64"
    blocked = kind == "solve" and rng.random() < 0.25
    lo, hi = (32, 640) if three_d else (64, 12000)
    tiles, dims = [], []
    side = math.exp(rng.uniform(math.log(lo), math.log(hi)))
    for _ in range(3 if three_d else 2):
        n = side * rng.uniform(0.7, 1.4)                    # not square
        t = min(rng.choice([1, 1, 2, 3, 4, 5, 8]), max(1, int(n) // (8 if three_d else 16)))
        w = max(1, int(n / t))
        if rng.random() < 0.5:
            w = max(2, w // 2 * 2)                           # half of the extents even, the others as they come
        tiles.append(t)
        dims.append(w * t)
    points = 1
    for n in dims:
        points *= n
    iters = every = 0
    if kind == "solve":
        iters = int(math.exp(rng.uniform(math.log(10), math.log(120))))
        iters = max(2, min(iters, int(MOST_UPDATES / points)))
        every = max(1, iters // rng.choice([1, 2, 4]))
    return _case(None, kind, dims, tiles, dtype, iters, every, rng.choice([4, 8, 12]) if blocked else 1)


def _field(case, seed):
    """Padded field: ring and interior uniform in [-1, 1)."""
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    shape = [n + 2 for n in _dims(case)]
    return torch.rand(shape, generator=gen, device="cuda", dtype=TORCH_TYPE[case["dtype"]]).mul_(2.0).sub_(1.0)


def prepare(case, seed):
    run_ = harness.JacobiRun(_dims(case), _tiles(case), NUMPY_NAME[case["dtype"]], tblock=case["tblock"])
    B.jacobi_prepare(run_.plan)
    field = _field(case, seed)
    norms = max(1, case["iters"] // case["every"] if case["every"] else 1)
    return {"run": run_, "case": case, "field": field, "out": torch.empty_like(field),
            "norms": torch.zeros(norms, dtype=torch.float64, device="cuda")}


def run(state):
    r, case = state["run"], state["case"]
    a, b, norms = r.a.data_ptr(), r.b.data_ptr(), state["norms"].data_ptr()
    stream = int(torch.cuda.current_stream().cuda_stream)
    B.jacobi_scatter(r.plan, state["field"].data_ptr(), a, stream)
    if case["kind"] == "check":
        B.halo_exchange(r.plan, a, stream)
        B.residual_norm(r.plan, a, norms, stream)
    else:
        a = B.jacobi_run(r.plan, a, b, case["iters"], case["every"], norms, stream)
    B.jacobi_gather(r.plan, a, state["out"].data_ptr(), stream)
    return {"field": state["out"], "norms": state["norms"]}


def work(case):
    """The field read once and written once; per point and iteration one update (3 or 5 additions, one product),
    per point and norm the difference, square and sum on top of the neighbours' sum."""
    points, padded = 1, 1
    for n in _dims(case):
        points *= n
        padded *= n + 2
    size = 8 if case["dtype"] == "f64" else 4
    per_update = 2 * len(_dims(case))
    norms = case["iters"] // case["every"] if case["every"] else 1
    return {"bytes": 2.0 * padded * size + 8.0 * norms,
            "flops": float(points) * (per_update * case["iters"] + (per_update + 3) * norms)}


def tolerance(case):
    """fp64: the update's order of additions is part of the library's contract, so fields agree to the bit and
    only the norms' sums may differ in order.  fp32: the field's rounding, against a computation in 64 bits."""
    return {"rel": 4e-15} if case["dtype"] == "f64" else {"rel": 4e-6}


def exact(case, seed):
    u = _field(case, seed).to(torch.float64)
    nd = u.dim()
    inner = tuple(slice(1, -1) for _ in range(nd))

    def shifted(d, by):
        n = u.shape[d]
        return u[tuple(slice(1 + by, n - 1 + by) if k == d else slice(1, -1) for k in range(nd))]

    def neighbours():
        s = shifted(nd - 1, -1) + shifted(nd - 1, 1)         # x, then y, then z: pairs of opposite neighbours
        pair = shifted(nd - 2, -1) + shifted(nd - 2, 1)
        s += pair
        if nd == 3:
            torch.add(shifted(0, -1), shifted(0, 1), out=pair)
            s += pair
        return s

    def norm():
        r = neighbours()
        r.sub_(u[inner], alpha=2.0 * nd)
        return float(r.square_().sum().sqrt())

    norms = []
    if case["kind"] == "check":
        norms.append(norm())
    scale = 0.25 if nd == 2 else 1.0 / 6.0
    for k in range(1, case["iters"] + 1):
        u[inner] = neighbours() * scale
        if case["every"] and k % case["every"] == 0:
            norms.append(norm())
    return {"field": u, "norms": torch.tensor(norms or [0.0], dtype=torch.float64)}
