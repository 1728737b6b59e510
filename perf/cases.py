"""What users of the planner have it do, as cases that can be timed.

A case is one call pattern through the package's entry points (Plan, Batch,
Engine) on a seeded maze: its kind, sizes and options as plain values.
listed() names the standing cases, draw() gives more of the same ranges,
prepare() makes what the calling program holds before the call, run() makes
the call once, work() says what the call cannot do without.

The mazes are the kinds the planner is measured on elsewhere in this
repository, made here with torch on the GPU from the case's seed: Bernoulli
obstacles, Bernoulli obstacles under filled rectangles, corridor mazes (depth
first search, 2% of the walls removed) and empty maps.  Sources and targets lie
on the largest 8-connected free component.

Every output is a whole number (int32 activity and path cells, int64 offsets),
so two versions of the planner agree only if they agree bit for bit.  Sizes and
numbers of targets follow from the case alone, the mazes from the seed; the
caller keeps buffers for the results, long enough for any seed's paths, and
the cells past the last path stay 0.
"""
import math
import random

import numpy as np
import torch

import paper_2004_00540_amd as omap

DEV = "cuda"


def _solve(name, maze, h, w, sources, targets, **more):
    """One maze through a Plan.  density: obstacle probability; layers: -1 for
    the run-time count; fresh: the plan is created and closed in the pass
    (else it is kept and the maze loaded into it); activity: the map is copied
    out; nearest: the source index of each path is asked for."""
    c = {"name": name, "kind": "solve", "maze": maze, "h": h, "w": w, "density": 0.35, "sources": sources,
         "targets": targets, "layers": -1, "schedule": 0, "fresh": False, "activity": True, "nearest": False}
    c.update(more)
    return c


def listed():
    return [
        # the smallest call: a 64 x 64 toy maze solved once, plan made for it
        _solve("toy_64", "bernoulli", 64, 64, 1, 4, density=0.30, fresh=True),
        # a street map of a city district, taxis as sources, the layer count
        # fixed, each customer's nearest taxi asked for (332 x 709, 33 taxis)
        _solve("taxis_332x709", "bernoulli", 332, 709, 33, 160, density=0.25, layers=160, nearest=True),
        # an ordinary map of odd sizes, solved again and again in a kept plan
        _solve("ragged_1021x1533", "bernoulli", 1021, 1533, 8, 512),
        # long corridors: a labyrinth where paths run for thousands of cells
        _solve("corridors_4096", "corridors", 4096, 4096, 1, 256),
        # the largest maze of the benchmark: 23170 x 23170 cells, 50,000 filled
        # rectangles over 40% noise, 16 sources, 4096 paths; the paths alone
        _solve("rectangles_23170", "rectangles", 23170, 23170, 16, 4096, density=0.40, activity=False),
        # an empty map and as many layers as its side, the method's own run
        # time figure: the map is what is wanted, default schedule ...
        _solve("empty_2000_fixed", "empty", 2000, 2000, 1, 16, density=0.0, layers=2000),
        # ... and the literal dense schedule, every tile in every round
        _solve("empty_2000_dense", "empty", 2000, 2000, 1, 16, density=0.0, layers=2000, schedule=omap.SCHEDULE_DENSE),
        # the largest map with sources everywhere: 26,000 x 26,000 cells, 5000
        # sources, 650 layers
        _solve("open_26000_5000src", "empty", 26000, 26000, 5000, 64, density=0.0, layers=650),
        # many uneven mazes at once: 512 with sides from 128 to 2048
        {"name": "batch_512", "kind": "batch", "mazes": 512, "side_lo": 128, "side_hi": 2048, "activity": False},
        # a serving engine on a burst of host-side queries
        {"name": "serve_20", "kind": "serve", "queries": 20, "side_lo": 256, "side_hi": 4096},
        # other path reconstructions on a propagated plan: random ties with the
        # nearest source of each path, and the Euclidean one
        {"name": "walk_random_2048", "kind": "walk", "mode": "random", "h": 2048, "w": 2048, "density": 0.35,
         "sources": 4, "targets": 2048, "nearest": True},
        {"name": "walk_euclid_2048", "kind": "walk", "mode": "euclidean", "h": 2048, "w": 2048, "density": 0.35,
         "sources": 4, "targets": 2048, "nearest": False},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng: random.Random):
    kind = rng.choice(["solve", "solve", "solve", "walk", "batch", "serve"])
    if kind == "batch":
        hi = _log_int(rng, 160, 2048)
        return {"kind": "batch", "mazes": _log_int(rng, 3, 512), "side_lo": rng.randint(64, 128), "side_hi": hi,
                "activity": hi <= 512 and rng.random() < 0.5}
    if kind == "serve":
        return {"kind": "serve", "queries": rng.randint(1, 20), "side_lo": rng.randint(64, 256),
                "side_hi": _log_int(rng, 300, 4096)}
    maze = rng.choice(["bernoulli", "bernoulli", "rectangles", "corridors", "empty"]) if kind == "solve" else "bernoulli"
    h = _log_int(rng, 32, {"corridors": 4096, "rectangles": 16000}.get(maze, 6000))
    w = _log_int(rng, max(32, h // 4), min(4 * h, {"corridors": 4096, "rectangles": 16000}.get(maze, 6000)))
    cells = h * w
    density = {"empty": 0.0, "rectangles": 0.40}.get(maze, round(rng.uniform(0.2, 0.38), 3))
    sources, targets = _log_int(rng, 1, min(64, 1 + cells // 64)), _log_int(rng, 1, min(4096, 1 + cells // 16))
    if kind == "walk":
        return {"kind": "walk", "mode": rng.choice(["random", "euclidean", "first_max"]), "h": h, "w": w,
                "density": density, "sources": sources, "targets": targets, "nearest": rng.random() < 0.5}
    c = _solve("", maze, h, w, sources, targets, density=density, fresh=rng.random() < 0.3,
               activity=rng.random() < 0.6, nearest=rng.random() < 0.3)
    del c["name"]
    if maze == "empty" or rng.random() < 0.25:
        c["layers"] = _log_int(rng, 8, 2 * max(h, w))
    if cells <= 1500 * 1500 and maze != "corridors":
        c["schedule"] = rng.choice([0, 0, omap.SCHEDULE_ACTIVE, omap.SCHEDULE_BITS, omap.SCHEDULE_DENSE])
    elif maze == "empty" and rng.random() < 0.5:
        c["sources"] = _log_int(rng, 64, 5000)
    return c


# ---- mazes ---------------------------------------------------------------------

def _components(free):
    """Labels (int32, flat cell index of a representative) of the 8-connected
    components of a bool grid: hook every label to its smallest neighbour's,
    then follow labels to their roots, until nothing changes."""
    H, W = free.shape
    none = H * W
    start = torch.arange(none, dtype=torch.int32, device=free.device).view(H, W)
    lab = torch.where(free, start, none)
    cells = free.flatten().nonzero().flatten()
    parent = torch.arange(none + 1, dtype=torch.int32, device=free.device)
    own = cells.to(torch.int32)
    while True:
        m = lab.clone()
        torch.minimum(m[:, 1:], lab[:, :-1], out=m[:, 1:])
        torch.minimum(m[:, :-1], lab[:, 1:], out=m[:, :-1])
        n = m.clone()
        torch.minimum(n[1:], m[:-1], out=n[1:])
        torch.minimum(n[:-1], m[1:], out=n[:-1])
        near = n.flatten()[cells]
        if bool((near == own).all()):
            return lab
        del m, n
        parent.scatter_reduce_(0, own.long(), near, "amin")
        while True:
            up = parent[own.long()]
            same = bool((up == own).all())
            own = up
            if same:
                break
        parent[cells] = own
        lab.view(-1)[cells] = own


def _rectangles(occ, n, lo, hi, gen):
    """Fill n rectangles with sides in [lo, hi] (corners in a difference grid,
    summed along both axes)."""
    H, W = occ.shape
    d = torch.zeros((H + 1, W + 1), dtype=torch.int32, device=DEV)
    r0 = torch.randint(0, H, (n,), generator=gen, device=DEV)
    c0 = torch.randint(0, W, (n,), generator=gen, device=DEV)
    r1 = (r0 + torch.randint(lo, hi + 1, (n,), generator=gen, device=DEV)).clamp(max=H)
    c1 = (c0 + torch.randint(lo, hi + 1, (n,), generator=gen, device=DEV)).clamp(max=W)
    one = torch.ones(n, dtype=torch.int32, device=DEV)
    for r, c, v in ((r0, c0, one), (r0, c1, -one), (r1, c0, -one), (r1, c1, one)):
        d.index_put_((r, c), v, accumulate=True)
    cover = d.cumsum(0, dtype=torch.int32).cumsum(1, dtype=torch.int32)
    occ |= (cover[:H, :W] > 0).to(torch.uint8)


def _dfs_block(n, rnd):
    """Passages of a depth-first-search maze on an n x n lattice: (open to the
    right, open downwards) of each lattice cell."""
    right, down, seen = bytearray(n * n), bytearray(n * n), bytearray(n * n)
    at = rnd.randrange(n * n)
    seen[at] = 1
    stack = [at]
    while stack:
        at = stack[-1]
        c = at % n
        todo = []
        if c + 1 < n and not seen[at + 1]:
            todo.append(at + 1)
        if c and not seen[at - 1]:
            todo.append(at - 1)
        if at + n < n * n and not seen[at + n]:
            todo.append(at + n)
        if at >= n and not seen[at - n]:
            todo.append(at - n)
        if not todo:
            stack.pop()
            continue
        to = todo[int(rnd.random() * len(todo))]
        (right if abs(to - at) == 1 else down)[min(at, to)] = 1
        seen[to] = 1
        stack.append(to)
    return [np.frombuffer(bytes(a), np.uint8).reshape(n, n).astype(bool) for a in (right, down)]


def _turned(right, down, flips, swap):
    if swap:
        right, down = down.T, right.T
    if flips & 1:   # left-right: a passage to the right belongs to the other cell
        right, down = np.roll(right[:, ::-1], -1, 1), down[:, ::-1]
    if flips & 2:
        right, down = right[::-1], np.roll(down[::-1], -1, 0)
    return right, down


def _corridors(H, W, rnd, blocks=4):
    """Corridor maze: depth-first-search blocks joined along every block edge
    at one place, 2% of the remaining walls removed."""
    h, w = (H + 1) // 2, (W + 1) // 2
    n = max(8, min(256, max(h, w)))
    pool = [_dfs_block(n, rnd) for _ in range(1 if n >= max(h, w) else blocks)]
    by, bx = -(-h // n), -(-w // n)
    right, down = np.zeros((by * n, bx * n), bool), np.zeros((by * n, bx * n), bool)
    for y in range(by):
        for x in range(bx):
            r, d = _turned(*pool[rnd.randrange(len(pool))], rnd.randrange(4), rnd.random() < 0.5)
            right[y * n:(y + 1) * n, x * n:(x + 1) * n] = r
            down[y * n:(y + 1) * n, x * n:(x + 1) * n] = d
            if x + 1 < bx:
                right[y * n + rnd.randrange(n), (x + 1) * n - 1] = True
            if y + 1 < by:
                down[(y + 1) * n - 1, x * n + rnd.randrange(n)] = True
    g = np.random.default_rng(rnd.randrange(1 << 30))
    right = (right | (g.random(right.shape, np.float32) < 0.02))[:h, :w]
    down = (down | (g.random(down.shape, np.float32) < 0.02))[:h, :w]
    occ = np.ones((2 * h, 2 * w), np.uint8)
    occ[0::2, 0::2] = 0
    occ[0::2, 1::2] = ~right
    occ[1::2, 0::2] = ~down
    return torch.from_numpy(np.ascontiguousarray(occ[:H, :W])).to(DEV)


def _obstacles(maze, h, w, density, gen, rnd):
    if maze == "corridors":
        return _corridors(h, w, rnd)
    if maze == "empty":
        return torch.zeros((h, w), dtype=torch.uint8, device=DEV)
    occ = (torch.rand((h, w), generator=gen, device=DEV) < density).to(torch.uint8)
    if maze == "rectangles":   # 50,000 with sides of 2 to 200 on 23170 x 23170 cells
        _rectangles(occ, max(1, round(50000 * h * w / 23170 ** 2)), 2, min(200, max(2, h // 2), max(2, w // 2)), gen)
    return occ


def _places(occs, wanted, gen):
    """For each maze n cells (row, col) of its largest component, as int32 host
    arrays: distinct, repeated only where the component is smaller.  The mazes
    are labelled on one sheet, in rows as wide as the widest, one wall apart."""
    width = max(max(o.shape[1] for o in occs), 8192 if len(occs) > 1 else 0)
    at, y, x, tall = [], 0, 0, 0
    for o in occs:
        if x and x + o.shape[1] > width:
            y, x, tall = y + tall + 1, 0, 0
        at.append((y, x))
        x, tall = x + o.shape[1] + 1, max(tall, o.shape[0])
    sheet = torch.zeros((y + tall, width), dtype=torch.bool, device=DEV)
    for o, (y, x) in zip(occs, at):
        sheet[y:y + o.shape[0], x:x + o.shape[1]] = o == 0
    lab = _components(sheet)
    size = torch.bincount(lab.flatten().masked_select(sheet.flatten()), minlength=sheet.numel() + 1)
    out = []
    for o, n, (y, x) in zip(occs, wanted, at):
        mine = lab[y:y + o.shape[0], x:x + o.shape[1]]
        roots = mine.masked_select(o == 0).long()
        if not roots.numel():
            o[0, 0] = 0
            out.append(np.zeros((n, 2), np.int32))
            continue
        best = roots[size[roots].argmax()].to(torch.int32)
        cells = (mine == best).flatten().nonzero().flatten()
        if cells.numel() <= 4 * n:
            cells = cells[torch.randperm(cells.numel(), generator=gen, device=DEV)[:n]]
        else:   # distinct by rejection: draw twice as many, keep the first of each
            pick = torch.randint(0, cells.numel(), (2 * n + 16,), generator=gen, device=DEV).cpu().numpy()
            _, first = np.unique(pick, return_index=True)
            cells = cells[torch.from_numpy(pick[np.sort(first)][:n]).to(DEV)]
        cells = np.resize(cells.cpu().numpy(), n)
        out.append(np.stack([cells // o.shape[1], cells % o.shape[1]], 1).astype(np.int32))
    return out


def _mazes(case, gen, rnd):
    """The mazes of a batch (Bernoulli, p in [0.2, 0.45], 1 to 8 sources, 16 to
    512 targets) or of a burst of queries (corridors or Bernoulli(0.35) by a
    coin, square, 1 to 16 sources, 8 to 2048 targets)."""
    serve = case["kind"] == "serve"
    occs, wanted, pool = [], [], {}
    for h, w, sources, targets, coin, p in _sizes(case):
        if serve and coin:
            hi = case["side_hi"]
            if not pool:
                pool["maze"] = _corridors(hi, hi, rnd, blocks=2)
            y, x = (2 * rnd.randint(0, (hi - h) // 2) for _ in range(2))
            occ = pool["maze"][y:y + h, x:x + w].contiguous()
        else:
            occ = _obstacles("bernoulli", h, w, p, gen, rnd)
        occs.append(occ)
        wanted.append(sources + targets)
    places = _places(occs, wanted, gen)
    return [(o, p[:z[2]].copy(), p[z[2]:].copy()) for o, p, z in zip(occs, places, _sizes(case))]


def _sizes(case):
    """(height, width, sources, targets, corridors, density) of each maze of a
    batch or burst, from the case alone."""
    serve = case["kind"] == "serve"
    lo, hi = case["side_lo"], case["side_hi"]
    rnd = random.Random("%s %d %d" % (case["kind"], lo, hi))
    out = []
    for _ in range(case["queries" if serve else "mazes"]):
        h, w = _log_int(rnd, lo, hi), _log_int(rnd, lo, hi)
        out.append((h, h if serve else w, rnd.randint(1, 16 if serve else 8),
                    rnd.randint(8, 2048) if serve else rnd.randint(16, 512),
                    serve and rnd.random() < 0.5, 0.35 if serve else rnd.uniform(0.2, 0.45)))
    return out


def _room(h, w, targets, winding=False, layers=-1):
    """Cells to keep for `targets` paths: none longer than a few times the
    maze's sides (corridors: many times), nor than its layers or its cells."""
    longest = min(h * w, (24 if winding else 3) * (h + w), layers + 1 if layers >= 0 else h * w)
    return min(targets * longest, 1 << 26)


# ---- the calls -------------------------------------------------------------------

def prepare(case, seed):
    gen = torch.Generator(device=DEV).manual_seed(seed)
    rnd = random.Random(seed)
    kind = case["kind"]
    state = dict(case=case, seed=seed)
    if kind == "batch":
        state["mazes"] = _mazes(case, gen, rnd)
        room = sum(_room(h, w, t) for h, w, _, t, _, _ in _sizes(case))
        state["cells"] = torch.zeros(min(room, 1 << 27), dtype=torch.int32, device=DEV)
        return state
    if kind == "serve":
        state["mazes"] = [(o.cpu().numpy(), s, t) for o, s, t in _mazes(case, gen, rnd)]
        state["engine"] = omap.Engine(2 << 30, max_slots=32)
        state["results"] = [(np.zeros(t, np.int32), np.zeros(t + 1, np.int64), np.zeros(_room(h, w, t, c), np.int32))
                            for h, w, _, t, c, _ in _sizes(case)]
        return state
    maze, h, w = case.get("maze", "bernoulli"), case["h"], case["w"]
    occ = _obstacles(maze, h, w, case["density"], gen, rnd)
    n = case["sources"] + case["targets"]
    if maze == "empty":
        m = min(h * w, 1 << 22)   # distinct cells, spread over the map
        pick = torch.randperm(m, generator=gen, device=DEV)[:n].cpu().numpy().astype(np.int64)
        pick = (np.resize(pick, n) * (h * w // m) + rnd.randrange(h * w)) % (h * w)
        places = np.stack([pick // w, pick % w], 1).astype(np.int32)
    else:
        places = _places([occ], [n], gen)[0]
        torch.cuda.empty_cache()
    state["occ"], state["src"], state["tgt"] = occ, places[:case["sources"]].copy(), places[case["sources"]:].copy()
    t = case["targets"]
    state["lengths"] = torch.empty(t, dtype=torch.int32, device=DEV)
    state["offsets"] = torch.empty(t + 1, dtype=torch.int64, device=DEV)
    state["cells"] = torch.zeros(_room(h, w, t, maze == "corridors", case.get("layers", -1)), dtype=torch.int32, device=DEV)
    if kind == "walk" or not case["fresh"]:
        state["plan"] = omap.Plan(occ, state["src"], state["tgt"], schedule=case.get("schedule", 0))
        if kind == "walk":
            state["plan"].propagate()
    return state


def _kept(paths, cells):
    """Paths with their cells copied to the caller's buffer."""
    cells[:len(paths[2])].copy_(paths[2])
    return paths[:2] + (cells,) + paths[3:]


def _solved(plan, case, state):
    info = plan.propagate(case["layers"], sync=case["activity"])
    if case["nearest"]:
        out = {"paths": _kept(plan.paths(source_index=True), state["cells"])}
    else:
        plan.extract_into(state["lengths"], state["offsets"], state["cells"])
        out = {"paths": (state["lengths"], state["offsets"], state["cells"])}
    if case["activity"]:
        out["activity"] = plan.activity()
        out["layers"], out["reached"] = info["layers"], info["reached_cells"]
    return out


def _served(engine, mazes, results):
    ids = {engine.submit(o, s, t): k for k, (o, s, t) in enumerate(mazes)}
    while ids:
        engine.step(rounds=4)
        for q in engine.completed():
            r = engine.fetch(q)
            lengths, offsets, cells = results[ids.pop(q)]
            lengths[:], offsets[:], cells[:len(r.cells)] = r.lengths, r.offsets, r.cells
    return results


def run(state):
    case = state["case"]
    if case["kind"] == "walk":
        return _kept(state["plan"].paths(mode=case["mode"], seed=state["seed"], source_index=case["nearest"]),
                     state["cells"])
    if case["kind"] == "batch":
        with omap.Batch(state["mazes"]) as b:
            infos = b.propagate(sync=case["activity"])
            out = {"paths": _kept(b.paths(), state["cells"])}
            if case["activity"]:
                out["layers"] = np.array([i["layers"] for i in infos])
                flat = torch.empty(sum(h * w for h, w in b.shapes), dtype=torch.int32, device=DEV)
                at = 0
                for i, (h, w) in enumerate(b.shapes):
                    b.activity(i, out=flat[at:at + h * w].view(h, w))
                    at += h * w
                out["activity"] = flat
        return out
    if case["kind"] == "serve":
        return _served(state["engine"], state["mazes"], state["results"])
    opts = {"schedule": case["schedule"]}
    if case["fresh"]:
        with omap.Plan(state["occ"], state["src"], state["tgt"], **opts) as plan:
            return _solved(plan, case, state)
    plan = state["plan"]
    plan.load(state["occ"], state["src"], state["tgt"])
    return _solved(plan, case, state)


def work(case):
    """Occupancy read once, the map written once where it is asked for, path
    cells written once (a path taken as a third of height + width, corridors
    twice that sum); one maximum over the 3 x 3 window per free cell."""
    kind = case["kind"]
    if kind in ("batch", "serve"):
        lo, hi = case["side_lo"], case["side_hi"]
        span = max(math.log(hi / lo), 1e-9)
        side, area = (hi - lo) / span, (hi * hi - lo * lo) / (2 * span)
        n, targets = (case["queries"], 1028) if kind == "serve" else (case["mazes"], 264)
        cells = n * (area if kind == "serve" else side * side)
        cells = max(cells, n * lo * lo)
        paths = n * targets * 2 * max(side, lo) / 3
        return {"bytes": cells * (5 if case.get("activity") else 1) + 4 * paths, "flops": 8 * 0.67 * cells}
    cells = case["h"] * case["w"]
    reach = (2 if case.get("maze") == "corridors" else 1 / 3) * (case["h"] + case["w"])
    paths = 4 * case["targets"] * min(reach, case.get("layers", -1) if case.get("layers", -1) > 0 else reach)
    if kind == "walk":   # each path cell's 3 x 3 window of the map, and the cell written
        return {"bytes": 10 * paths, "flops": 8 * paths / 4}
    return {"bytes": cells + (4 * cells if case["activity"] else 0) + paths, "flops": 8 * (1 - case["density"]) * cells}


def exact(case, seed):
    """The activity map and counts of a smaller maze from breadth-first layers
    in float64 (a maximum over the 3 x 3 window each); the paths, whole numbers
    that follow from the map by a rule, have no value here."""
    if case["kind"] != "solve" or not case["activity"] or case["h"] * case["w"] > 2_000_000 or case["maze"] == "corridors":
        return None
    s = prepare(dict(case, fresh=True), seed)
    free = (s["occ"] == 0).double()
    seen = torch.zeros_like(free)
    seen[s["src"][:, 0], s["src"][:, 1]] = 1
    total, n, count = torch.zeros_like(free), 0, int(seen.sum())
    while case["layers"] < 0 or n <= case["layers"]:
        total += seen           # cells at distance d are in the layers d, d+1, ...
        more = torch.nn.functional.max_pool2d(seen[None], 3, 1, 1)[0] * free
        n += 1
        if case["layers"] < 0:
            c = int(more.sum())
            if c == count:
                break
            count = c
        seen = more
    reached = int((total > 0).sum())
    return {"paths": [None] * (4 if case["nearest"] else 3), "activity": total.long(), "layers": n - 1, "reached": reached}
