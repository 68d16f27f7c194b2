"""Timed cases of the matching library: what its users have it do, through the
package's public entry points, from the smallest call to a whole batch.

listed() names the cases, draw(rng) gives more of the same ranges, prepare()
makes what a program holds before the call (device-resident point sets, a
context, a plan), run() makes one pass, work() states the bytes and operations
a pass cannot do without, exact() gives the same outputs in 64 bits from plain
torch.  The inputs are seeded stand-ins for interest points of videos: uniform
positions, non-negative L1-normalised descriptors of length 162, models with
increasing frames, scenes sorted by frame that hold jittered copies of the
models.
"""
import math

import numpy as np
import torch

import paper_1505_00581_amd as stm
from paper_1505_00581_amd import synth

DIM = 162
L1, L2, L3 = 0.6, 0.2, 5.0  # the energy weights every case uses
LANE_OPS = 11               # lane operations of one relaxation of the recursion


def listed():
    return [
        # the plain exact workload of the tests: a first call, a short clip; latency and launches count
        dict(name="match_small", kind="match", M=20, frames=100, per_frame=4, W=2, K=16, T=10, unary="f32",
             dummy=-1.0, reading="frames"),
        # one model looked for at every offset of a video: the everyday call
        dict(name="match_model", kind="match", M=75, frames=1500, per_frame=20, W=3, K=64, T=10, unary="f32",
             dummy=-1.0, reading="frames"),
        # the same with the split-precision appearance table, a long model, lists of odd length
        dict(name="match_bf16", kind="match", M=99, frames=1201, per_frame=17, W=3, K=57, T=10, unary="bf16",
             dummy=-1.0, reading="frames"),
        # points may stay unmatched (occlusion)
        dict(name="match_dummy", kind="match", M=60, frames=1500, per_frame=20, W=3, K=64, T=10, unary="f32",
             dummy=0.5, reading="frames"),
        # a model with up to three points per frame, split into chains
        dict(name="chains", kind="chains", model_frames=75, frames=1500, per_frame=20, W=3, K=64, n_chains=3),
        # the benchmark: ten models against one video in one replayed plan
        dict(name="plan_scene", kind="plan", models=10, m_lo=50, m_hi=100, scenes=1, f_lo=1500, f_hi=1500, p_lo=20,
             p_hi=20, K=64, W=3, density=False),
        # many models against several videos of uneven density, lists capped by density
        dict(name="plan_uneven", kind="plan", models=16, m_lo=30, m_hi=150, scenes=4, f_lo=500, f_hi=3000, p_lo=10,
             p_hi=30, K=64, W=3, density=True),
        # streaming: fifty models against every block of sixty points of a sparse video
        dict(name="blocks", kind="blocks", models=50, M=30, frames=723, points=754, block=60, T=10),
        # the same video as one trellis, fifty models, closeness limit ten
        dict(name="trellis_t10", kind="trellis", models=50, M=30, frames=723, points=754, T=10),
        # one model without a closeness limit
        dict(name="trellis_open", kind="trellis", models=1, M=30, frames=723, points=754, T=0),
        # lists cut by the learned score before the exact recursion
        dict(name="pruned_match", kind="pruned", M=75, frames=1500, per_frame=20, W=3, K=64, topk=48),
        # forward and backward of the score network on one training batch
        dict(name="pruner_grad", kind="grad", M=75, frames=1500, per_frame=20, W=3, K=64, groups=1024),
    ]


def draw(rng):
    def logint(lo, hi):
        return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))

    kind = rng.choice(["match", "match", "match", "chains", "plan", "blocks", "trellis", "trellis", "pruned", "grad"])
    if kind == "match":
        M = logint(5, 150)
        sparse = rng.random() < 0.25
        c = dict(kind=kind, M=M, frames=max(logint(60, 3000), 4 * M + 1),
                 per_frame=rng.randint(1, 3) if sparse else rng.randint(4, 30),
                 W=rng.randint(8, 20) if sparse else rng.randint(1, 4), K=logint(4, 64), T=rng.choice([0, 5, 8, 10, 10]),
                 unary=rng.choice(["f32", "f32", "bf16"]), dummy=-1.0, reading="frames")
        form = rng.random()
        if form < 0.2:
            c["dummy"] = rng.choice([0.16, 0.5, 1.0])
        elif form < 0.4:
            c["reading"] = rng.choice(["span", "unsigned", "node"])
        return c
    if kind == "chains":
        n = logint(10, 90)
        return dict(kind=kind, model_frames=n, frames=max(logint(100, 1500), 3 * n), per_frame=rng.randint(6, 20),
                    W=rng.randint(2, 3), K=logint(8, 64), n_chains=rng.randint(2, 3))
    if kind == "plan":
        models, scenes = logint(1, 12), rng.randint(1, 3)
        m_hi = rng.randint(30, 120)
        f_hi = rng.randint(400, 1800)
        p_hi = rng.randint(8, 28)
        return dict(kind=kind, models=models, m_lo=rng.randint(12, m_hi), m_hi=m_hi, scenes=scenes,
                    f_lo=rng.randint(300, f_hi), f_hi=f_hi, p_lo=rng.randint(6, p_hi), p_hi=p_hi,
                    K=rng.randint(24, 64), W=rng.randint(2, 3), density=rng.random() < 0.5)
    if kind == "blocks":
        frames = logint(150, 723)
        return dict(kind=kind, models=logint(1, 50), M=rng.randint(12, 40), frames=frames,
                    points=frames + rng.randint(0, frames // 2), block=rng.randint(32, 64), T=rng.choice([6, 10, 15]))
    if kind == "trellis":
        frames = logint(60, 723)
        return dict(kind=kind, models=logint(1, 50), M=rng.randint(8, 40), frames=frames,
                    points=frames + rng.randint(0, frames // 10), T=rng.choice([0, 6, 10, 10, 20]))
    if kind == "pruned":
        M = logint(10, 100)
        return dict(kind=kind, M=M, frames=max(logint(100, 1500), 3 * M), per_frame=rng.randint(8, 24), W=3, K=64,
                    topk=rng.randint(12, 56))
    M = logint(10, 100)
    return dict(kind=kind, M=M, frames=max(logint(100, 1500), 3 * M), per_frame=rng.randint(6, 24), W=rng.randint(2, 3),
                K=rng.randint(24, 64), groups=logint(64, 2048))


# ---- inputs -------------------------------------------------------------------------

class _Set:
    """A point set: xy [n, 2] float32 and t [n] int32 (numpy), desc [n, DIM] float32 (GPU)."""

    def __init__(self, xy, t, desc, n_frames=0):
        self.xy, self.t, self.desc, self.n_frames = xy.astype(np.float32), t.astype(np.int32), desc, n_frames

    def device(self):
        return stm.DevicePoints(torch.from_numpy(self.xy).cuda(), torch.from_numpy(self.t).cuda(), self.desc,
                                self.n_frames)


def _descriptors(gen, n):
    g = torch.randn((n, DIM), generator=gen, device="cuda", dtype=torch.float32).square_()
    return g / g.sum(1, keepdim=True)


def _model_frames(rng, m, hi, T):
    """m increasing frames from 0 to hi, gaps below T (the same span for every seed)."""
    while True:
        f = np.sort(np.concatenate([[0, hi], 1 + rng.choice(hi - 1, size=m - 2, replace=False)]))
        if T <= 0 or int(np.diff(f).max()) < T:
            return f.astype(np.int32)


def _model(rng, gen, m, size, T, hi=None):
    t = _model_frames(rng, m, hi if hi is not None else int(math.ceil(1.5 * m)), T)
    return _Set(rng.uniform(0, 1, (m, 2)) * size, t, _descriptors(gen, m))


def _scene(rng, gen, models, counts, size, copies):
    """Uniform clutter, counts[f] points in frame f, and jittered copies of the models, sorted by (frame, x)."""
    F, n = len(counts), int(counts.sum())
    xy, t, d = [rng.uniform(0, 1, (n, 2)) * size], [np.repeat(np.arange(F), counts)], [_descriptors(gen, n)]
    for m in models:
        for _ in range(copies):
            tau = int(rng.integers(0, F - int(m.t[-1])))
            c = m.xy.astype(np.float64).mean(0)
            xy.append((m.xy - c) * rng.uniform(0.9, 1.1) + rng.uniform(0, 1, 2) * size + rng.normal(0, 3, m.xy.shape))
            t.append(np.clip(tau + m.t + np.rint(rng.normal(0, 1, m.t.shape)), 0, F - 1))
            g = (m.desc + 0.02 * torch.randn(m.desc.shape, generator=gen, device="cuda")).clamp_(min=0)
            d.append(g / g.sum(1, keepdim=True))
    xy, t = np.concatenate(xy).astype(np.float32), np.concatenate(t).astype(np.int32)
    order = np.lexsort((xy[:, 0], t))
    return _Set(xy[order], t[order], torch.cat(d)[torch.from_numpy(order).cuda()].contiguous(), F)


def _inputs(c, seed):
    """(models, scenes, saliency) of a case, from the seed alone."""
    rng = np.random.default_rng([seed, 11])
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    wide, narrow = np.array([320.0, 240.0]), np.array([160.0, 120.0])
    k = c["kind"]
    if k in ("match", "pruned", "grad"):
        T = c.get("T", 10)
        m = _model(rng, gen, c["M"], wide, T if T > 0 else 10)
        return [m], [_scene(rng, gen, [m], np.full(c["frames"], c["per_frame"]), wide, 3)], None
    if k == "chains":
        ft = _model_frames(rng, c["model_frames"], int(math.ceil(1.5 * c["model_frames"])), 10)
        per = np.full(c["model_frames"], c["n_chains"])
        per[2::5], per[4::5] = 1, 2  # some frames hold fewer points
        t = np.repeat(ft, per)
        m = _Set(rng.uniform(0, 1, (len(t), 2)) * wide, t, _descriptors(gen, len(t)))
        s = _scene(rng, gen, [m], np.full(c["frames"], c["per_frame"]), wide, 3)
        return [m], [s], rng.uniform(0, 1, len(t)).astype(np.float32)
    if k == "plan":
        span = (lambda lo, hi, n: np.linspace(lo, hi, n).round().astype(int))  # uneven, the same for every seed
        models = [_model(rng, gen, int(x), wide, 10) for x in span(c["m_lo"], c["m_hi"], c["models"])]
        scenes = []
        for f in span(c["f_lo"], c["f_hi"], c["scenes"]):
            counts = rng.integers(c["p_lo"], c["p_hi"] + 1, int(f))
            scenes.append(_scene(rng, gen, models, counts, wide, 5 if c["scenes"] == 1 else 1))
        return models, scenes, None
    # the sparse video: about one point per frame, copies of up to five models
    models = [_model(rng, gen, c["M"], narrow, 10 if c["T"] == 0 else min(10, c["T"]), hi=int(1.5 * c["M"]))
              for _ in range(c["models"])]
    copies = min(5, c["models"], c["points"] // (4 * c["M"]))
    counts = rng.multinomial(c["points"] - c["M"] * copies, np.full(c["frames"], 1.0 / c["frames"]))
    return models, [_scene(rng, gen, models[:copies], counts, narrow, 1)], None


def _params(c):
    k = c["kind"]
    p = synth.Params(lambda1=L1, lambda2=L2, lambda3=L3, T=c.get("T", 10), window=c.get("W", 0),
                     k_max=c["block"] if k == "blocks" else c.get("K", 1), k_density=c.get("density", False))
    if k == "match":
        p.unary_bf16 = c["unary"] == "bf16"
        p.w_dummy = c["dummy"] if c["dummy"] >= 0 else None
        p.closeness_span, p.angle_unsigned, p.causal_node = (c["reading"] == x for x in ("span", "unsigned", "node"))
    return p


def _n_blocks(c, models, scene):
    return max(1, min(scene.n_frames - int(max(m.t[-1] for m in models)), len(scene.t) - c["block"] + 1))


def _groups(c, model, scene, seed):
    """Training groups (offset, point) and label nodes: a uniform draw from each list."""
    rng = np.random.default_rng([seed, 13])
    n = scene.n_frames - int(model.t[-1])
    g = np.stack([rng.integers(0, n, c["groups"]), rng.integers(0, c["M"], c["groups"])], 1).astype(np.int32)
    lists, count = _frame_lists(scene, c["W"], c["K"], False)
    f = g[:, 0] + model.t[g[:, 1]]
    pick = (rng.uniform(0, 1, c["groups"]) * count[f]).astype(np.int64)
    return g, lists[f, pick].astype(np.int32)


def prepare(case, seed):
    c = case
    models, scenes, sal = _inputs(c, seed)
    ctx = stm.Context(0)
    s = dict(case=c, ctx=ctx, params=_params(c), models=[m.device() for m in models],
             scenes=[x.device() for x in scenes])
    k = c["kind"]
    if k == "chains":
        s["saliency"] = torch.from_numpy(sal).cuda()
    elif k == "plan":
        pairs = np.array([(i, j) for i in range(c["models"]) for j in range(c["scenes"])], np.int32)
        s["plan"] = stm.Plan(ctx, s["models"], s["scenes"], pairs, s["params"])
        s["out"] = s["plan"].outputs()
    elif k == "blocks":
        pairs = np.array([(i, 0) for i in range(c["models"])], np.int32)
        plan = stm.Plan(ctx, s["models"], s["scenes"], pairs, s["params"])
        n, b = _n_blocks(c, models, scenes[0]), c["block"]
        cands, counts = [], []
        for q in range(c["models"]):  # a plan row past the last block gets empty lists
            rows = int(plan.row_offsets[q + 1] - plan.row_offsets[q])
            nodes = torch.arange(b, dtype=torch.int32, device="cuda") + torch.arange(n, dtype=torch.int32,
                                                                                     device="cuda")[:, None]
            cand = torch.zeros((rows, c["M"], b), dtype=torch.int32, device="cuda")
            cand[:n] = nodes[:, None, :]
            cnt = torch.zeros((rows, c["M"]), dtype=torch.int32, device="cuda")
            cnt[:n] = b
            cands.append(cand)
            counts.append(cnt)
        s.update(plan=plan, cands=cands, counts=counts, out=plan.outputs())
    elif k == "trellis":
        s["trellis"] = stm.Trellis(ctx, s["models"], s["scenes"][0], s["params"])
    elif k in ("pruned", "grad"):
        s["pruner"] = stm.Pruner(ctx, DIM)
        s["pruner"].set_params(synth.pruner_init(DIM, seed % 1000))
        s["pruner"].set_rule(stm.Pruner.FRAMES_FIRST)
        if k == "grad":
            s["groups"], s["labels"] = _groups(c, models[0], scenes[0], seed)
    return s


def _tensors(out):
    return {k: v for k, v in out.items() if torch.is_tensor(v)}


def run(state):
    s = state
    k = s["case"]["kind"]
    if k == "match":
        return _tensors(s["ctx"].match(s["models"][0], s["scenes"][0], s["params"]))
    if k == "chains":
        return _tensors(s["ctx"].match_chains(s["models"][0], s["scenes"][0], s["params"], s["saliency"],
                                              s["case"]["n_chains"]))
    if k == "plan":
        return _tensors(s["plan"].run(s["out"]))
    if k == "blocks":
        return _tensors(s["plan"].run_lists(s["cands"], s["counts"], s["case"]["block"], s["out"]))
    if k == "trellis":
        return _tensors(s["trellis"].run())
    if k == "pruned":
        return _tensors(s["pruner"].match(s["models"][0], s["scenes"][0], s["params"], topk=s["case"]["topk"]))
    loss, grad, scores = s["pruner"].gradient(s["models"][0], s["scenes"][0], s["params"], s["groups"], s["labels"])
    return dict(loss=np.array([loss], np.float32), grad=grad, scores=scores)


# ---- the work of a pass ---------------------------------------------------------------

def _window_relaxations(M, n_tau, per_frame, W, K, T):
    """Expected feasible relaxations of n_tau windowed matchings: lists of the first K of per_frame points in each
    frame, nearest frames first, consecutive points 1..T-1 frames apart, model gaps of mean 1.5."""
    have, left = {}, float(K)
    for s in range(2 * W + 1):
        d = 0 if s == 0 else (-((s + 1) // 2) if s % 2 else s // 2)
        have[d] = min(float(per_frame), left)
        left -= have[d]
    gaps = [(g, (2 / 3) * (1 / 3) ** (g - 1)) for g in range(1, 6)]
    lim = T if T > 0 else 1 << 30
    ok = {(a, b): sum(w for g, w in gaps if 0 < g + b - a < lim) for a in have for b in have}
    per_step = sum(have[a] * have[b] * have[e] * ok[a, b] * ok[b, e] for a in have for b in have for e in have)
    return n_tau * (M - 2) * per_step


def work(case):
    c, k = case, case["kind"]
    if k in ("blocks", "trellis"):
        pts = c["points"]
        reach = c["T"] - 1 if c["T"] > 0 else c["frames"]
        span = c["block"] if k == "blocks" else pts
        rho = pts / c["frames"]
        pos = np.arange(span) / rho  # expected frame of each node of the list
        fwd = np.minimum(reach, pos[-1] - pos) * rho
        back = np.minimum(reach, pos) * rho
        relax = float((fwd * back).sum()) * (c["M"] - 2) * c["models"]
        inputs = 4.0 * (pts * (DIM + 3) + c["models"] * c["M"] * (DIM + 3))
        if k == "trellis":
            return dict(bytes=inputs + c["models"] * (20.0 + 4 * c["M"]), flops=LANE_OPS * relax)
        n = max(1, min(c["frames"] - int(1.5 * c["M"]), pts - c["block"] + 1))
        lists = 4.0 * c["models"] * n * c["M"] * (c["block"] + 1)
        return dict(bytes=inputs + lists + c["models"] * n * (20.0 + 4 * c["M"]), flops=LANE_OPS * relax * n)
    if k == "plan":
        sizes = np.linspace(c["m_lo"], c["m_hi"], c["models"]).round()
        frames = np.linspace(c["f_lo"], c["f_hi"], c["scenes"]).round()
        pf = (c["p_lo"] + c["p_hi"]) / 2
        K = c["K"] if not c["density"] else min(c["K"], max(8, int((56 * 3 * pf - 1170) // 60)))
        fl = by = 4.0 * float(sizes.sum()) * (DIM + 3)
        for f in frames:
            by += 4.0 * f * pf * (DIM + 3)
            for m in sizes:
                n = max(0.0, f - 1.5 * m)
                by += n * (20.0 + 4 * m)
                fl += LANE_OPS * _window_relaxations(m, n, pf, c["W"], K, 10)
        return dict(bytes=by, flops=fl)
    M = 2.5 * c["model_frames"] if k == "chains" else c["M"]
    S = c["frames"] * c["per_frame"]
    inputs = 4.0 * (S + M) * (DIM + 3)
    if k == "grad":
        rows = 64.0 * c["groups"]
        params = 128 * (2 * DIM + 8) + 128 + 128 * 128 + 128 + 128 + 1
        return dict(bytes=inputs + 8.0 * params + 4.0 * rows,
                    flops=2.0 * rows * (2 * 128 * (2 * DIM + 8) + 3 * 128 * 128))
    span = 1.5 * (c["model_frames"] if k == "chains" else M)
    n = max(1.0, c["frames"] - span)
    K = c["topk"] if k == "pruned" else c["K"]
    fl = LANE_OPS * _window_relaxations(M, n, c["per_frame"], c["W"], K, c.get("T", 10)) + 3.0 * DIM * M * S
    if k == "pruned":
        fl += 2.0 * n * M * 64 * (128 * 128 + 8 * 128)
    return dict(bytes=inputs + n * (20.0 + 4 * M), flops=fl)


# ---- the same in 64 bits ------------------------------------------------------------------

def _frame_lists(scene, W, K, density):
    """The candidates of a point searched around frame f: nodes within W frames, the first K by (distance, node),
    ascending.  lists [F, K] (padded with 0) and count [F]."""
    t, F = scene.t, scene.n_frames
    start = np.searchsorted(t, np.arange(F + 1))
    lists, count = np.zeros((F, K), np.int64), np.zeros(F, np.int64)
    for f in range(F):
        lo, hi = start[max(f - W, 0)], start[min(f + W + 1, F)]
        nodes = np.arange(lo, hi)
        cap = K
        if density:
            rho = int(start[min(f + 2, F)] - start[max(f - 1, 0)])
            cap = min(K, max(8, min(64, (56 * rho - 1170) // 60)))
        keep = np.sort(nodes[np.lexsort((nodes, np.abs(t[lo:hi] - f)))][:cap])
        lists[f, :len(keep)], count[f] = keep, len(keep)
    return lists, count


def _turn(p, q):
    """Direction of q - p in turns."""
    d = q - p
    return torch.atan2(d[..., 1], d[..., 0]) / (2 * math.pi)


def _model_turns(m):
    """Angles (at i-1 and at i) of the model triangle ending at each point, in turns."""
    p = torch.from_numpy(m.xy.astype(np.float64)).cuda()
    a, b, e = p[2:], p[1:-1], p[:-2]
    z = torch.zeros(2, dtype=torch.float64, device="cuda")
    wrap = (lambda x: x - x.round())
    return torch.cat([z, wrap(_turn(b, e) - _turn(b, a))]), torch.cat([z, wrap(_turn(a, e) - _turn(a, b))])


def _distances(m, s, bf16):
    f, g = m.desc, s.desc
    if bf16:
        f, g = f.bfloat16(), g.bfloat16()
    f, g = f.double(), g.double()
    return torch.stack([(g - row).square().sum(1).sqrt() for row in f])


def _solve(m, s, cand, count, T, dummy=-1.0, reading="frames", bf16=False):
    """Optimum, its energy with the FP32 descriptors' distances and the appearance part of it, for every row of
    cand [n, M, K] (nodes, ascending, the first count [n, M] valid): the recursion of the energy in 64 bits."""
    INF = float("inf")
    n, M, K = cand.shape
    U = _distances(m, s, bf16)
    U32 = _distances(m, s, False) if bf16 else U
    sxy, st = torch.from_numpy(s.xy.astype(np.float64)).cuda(), torch.from_numpy(s.t.astype(np.int64)).cuda()
    mid, end = _model_turns(m)
    mt = [int(x) for x in m.t]
    w = L2 * L3 * 2 * math.pi
    span_T = T if reading == "span" and T > 0 else 0
    pair_T = 0 if span_T else T
    uns, node, dum = reading == "unsigned", reading == "node", dummy >= 0
    cw = L1 * max(dummy, 0.0)
    E, E32, EU = (torch.empty(n, dtype=torch.float64, device="cuda") for _ in range(3))
    slot = torch.arange(K, device="cuda")
    step_rows = max(1, (1 << 23) // K ** 3)
    for n0 in range(0, n, step_rows):
        cd, ok = cand[n0:n0 + step_rows], slot < count[n0:n0 + step_rows, :, None]
        B = cd.shape[0]
        at = torch.arange(B, device="cuda")
        X, F = sxy[cd], st[cd]
        u = [L1 * U[i][cd[:, i]] for i in range(M)]

        def pair(i):  # phi, admissible and |dt| of (point i-1, point i)
            x, y = X[:, i - 1, :, None], X[:, i, None]
            a, b = F[:, i - 1, :, None], F[:, i, None]
            good = (cd[:, i - 1, :, None] < cd[:, i, None]) if node else (a < b)
            if pair_T > 0:
                good = good & (b - a < pair_T)
            good = good & ok[:, i - 1, :, None] & ok[:, i, None]
            return _turn(x, y), good, ((mt[i] - mt[i - 1]) - (b - a)).abs().double()

        def terms(i, phi, new, C, V, r=None, col=None):  # V + w D^g, [B, k, r, c] or along (r, c) of each row
            if r is None:
                A, Nw, Cc, Vv = phi[:, :, :, None], new[:, None], C[:, :, None, :], V[:, :, :, None]
            else:
                A, Nw, Cc, Vv = phi[at, :, r], new[at, r, col][:, None], C[at, :, col], V[at, :, r]
            z1 = A + (0.5 - Nw if uns else 0.5 - Nw - mid[i])
            z1 -= z1.round()
            z2 = Cc - (Nw if uns else Nw + end[i])
            z2 -= z2.round()
            if uns:
                z1, z2 = z1.abs_().sub_(mid[i].abs()), z2.abs_().sub_(end[i].abs())
            z2 = z2.square_()
            return z1.square_().add_(z2).sqrt_().mul_(w).add_(Vv)

        phi, good, dt = pair(1)
        V = (u[0][:, :, None] + u[1][:, None] + L2 * dt).masked_fill_(~good, INF)
        inf1 = torch.full((B, K), INF, dtype=torch.float64, device="cuda")
        de = (cw + u[1]).masked_fill(~ok[:, 1], INF) if dum else inf1
        df = (u[0] + cw).masked_fill(~ok[:, 0], INF) if dum else inf1
        dg = torch.full((B,), 2 * cw if dum else INF, dtype=torch.float64, device="cuda")
        kept = [None, (V, phi, de, df, dg)]
        Cs = [None, None]
        for i in range(2, M):
            new, good, dt = pair(i)
            C = _turn(X[:, i - 2, :, None], X[:, i, None])
            if span_T:  # a triangle's first and last frames
                far = F[:, i, None] - F[:, i - 2, :, None] >= span_T
                C = C.masked_fill(far, INF)
                full = terms(i, phi, new, torch.where(far, 0.0, C), V)
                best = full.masked_fill_(far[:, :, None, :], INF).amin(1)
            else:
                best = terms(i, phi, new, C, V).amin(1)
            col_min = V.amin(1)
            if dum:
                best = torch.minimum(best, de[:, :, None])
            nv = (best + u[i][:, None] + (2 if i <= M - 2 else 1) * L2 * dt).masked_fill_(~good, INF)
            if dum:
                m_prev = torch.minimum(dg, df.amin(1))
                df2 = (cw + torch.minimum(de, col_min)).masked_fill(~ok[:, i - 1], INF)
                de = (u[i] + m_prev[:, None]).masked_fill(~ok[:, i], INF)
                dg, df = cw + m_prev, df2
            V, phi = nv, new
            kept.append((V, phi, de, df, dg))
            Cs.append(C)
        # the optimum: index K is the dummy on either side
        full = torch.cat([torch.cat([V, df[:, :, None]], 2), torch.cat([de, dg[:, None]], 1)[:, None]], 1)
        e, idx = full.reshape(B, -1).min(1)
        r, c = idx // (K + 1), idx % (K + 1)
        path = [c, r]
        for i in range(M - 1, 1, -1):
            V, phi, de, df, dg = kept[i - 1]
            new, C = kept[i][1], Cs[i]
            rr, cc = r.clamp(max=K - 1), c.clamp(max=K - 1)
            row_ok = V[at, :, rr]  # +inf where inadmissible
            if span_T:
                t = terms(i, phi, new, torch.where(C.isinf(), 0.0, C), V, rr, cc).masked_fill(C[at, :, cc].isinf(), INF)
            else:
                t = terms(i, phi, new, C, V, rr, cc)
            t = torch.where((c == K)[:, None], row_ok, t)
            t = torch.where((r == K)[:, None], df, t)
            eps = torch.where(r == K, dg, de[at, rr])
            k = torch.cat([t, eps[:, None]], 1).argmin(1)
            path.append(k)
            r, c = k, r
        path = torch.stack(path[::-1], 1)  # [B, M]
        dummies = path == K
        nodes = torch.gather(cd, 2, path.clamp(max=K - 1)[:, :, None])[:, :, 0]
        rows = torch.arange(M, device="cuda")
        a = torch.where(dummies, max(dummy, 0.0), U[rows, nodes]).sum(1) * L1
        a32 = torch.where(dummies, max(dummy, 0.0), U32[rows, nodes]).sum(1) * L1
        E[n0:n0 + B] = e
        E32[n0:n0 + B] = torch.where(e.isinf(), e, e - a + a32)
        EU[n0:n0 + B] = torch.where(e.isinf(), e, a32)
    return E, E32, EU


def _window_cands(m, s, W, K, density, tau0, n):
    lists, count = _frame_lists(s, W, K, density)
    f = tau0 + np.arange(n)[:, None] + (m.t - m.t[0])[None]
    return torch.from_numpy(lists[f]).cuda(), torch.from_numpy(count[f]).cuda()


def _solve_trellis(m, s, T):
    """The optimum over every node of the scene, and the energies of its assignment: rows of V by first node."""
    INF = float("inf")
    N, M = len(s.t), len(m.t)
    U = _distances(m, s, False)
    x = torch.from_numpy(s.xy.astype(np.float64)).cuda()
    t = torch.from_numpy(s.t.astype(np.int64)).cuda()
    phi = _turn(x[:, None], x[None])  # [first, second]
    dt = (t[None] - t[:, None]).double()
    bad = (dt <= 0) | (dt >= T) if T > 0 else dt <= 0
    mid, end = _model_turns(m)
    w = L2 * L3 * 2 * math.pi
    lo = np.searchsorted(s.t, s.t - T + 1) if T > 0 else np.zeros(N, np.int64)

    def cost(i, V, k0, r, rows):  # terms of predecessors k0.. (rows of them), middle nodes r, every last node
        z1 = phi[k0:rows, r, None] + (0.5 - phi[None, r] - mid[i])
        z1 -= z1.round()
        z2 = phi[k0:rows, None, :] - (phi[None, r] + end[i])
        z2 -= z2.round()
        return z1.square_().add_(z2.square_()).sqrt_().mul_(w).add_(V[k0:rows, r, None])

    V = (L1 * (U[0][:, None] + U[1][None]) + L2 * ((int(m.t[1]) - int(m.t[0])) - dt).abs()).masked_fill(bad, INF)
    kept = [None, V]
    for i in range(2, M):
        q = L1 * U[i][None] + (2 if i <= M - 2 else 1) * L2 * ((int(m.t[i]) - int(m.t[i - 1])) - dt).abs()
        best = torch.full((N, N), INF, dtype=torch.float64, device="cuda")
        for r0 in range(0, N, 16):
            r1 = min(N, r0 + 16)
            if r1 > 1:
                best[r0:r1] = cost(i, V, int(lo[r0]), slice(r0, r1), r1).amin(0)
        V = (best + q).masked_fill(bad, INF)
        kept.append(V)
    e, idx = V.reshape(-1).min(0)
    if not torch.isfinite(e):
        return e, e, e
    r, c = int(idx) // N, int(idx) % N
    path = [c, r]
    for i in range(M - 1, 1, -1):
        k = int(cost(i, kept[i - 1], 0, slice(r, r + 1), N)[:, 0, c].argmin())
        path.append(k)
        r, c = k, r
    a = L1 * sum(U[i][path[M - 1 - i]] for i in range(M))
    return e, e, a


def _exact_grad(c, m, s, seed):
    """Loss, gradient and scores of the training groups."""
    groups, labels = _groups(c, m, s, seed)
    lists, count = _frame_lists(s, c["W"], c["K"], False)
    U = _distances(m, s, False)
    G, M = len(groups), len(m.t)
    tau, i = torch.from_numpy(groups[:, 0].astype(np.int64)).cuda(), torch.from_numpy(groups[:, 1].astype(np.int64)).cuda()
    mt, st = torch.from_numpy(m.t.astype(np.int64)).cuda(), torch.from_numpy(s.t.astype(np.int64)).cuda()
    mx, sx = torch.from_numpy(m.xy.astype(np.float64)).cuda(), torch.from_numpy(s.xy.astype(np.float64)).cuda()
    lists, count = torch.from_numpy(lists).cuda(), torch.from_numpy(count).cuda()
    INF = float("inf")

    def cands(j):
        f = tau + mt[j] - mt[0]
        nodes = torch.zeros((G, 64), dtype=torch.int64, device="cuda")
        nodes[:, :lists.shape[1]] = lists[f]
        ok = torch.arange(64, device="cuda") < count[f][:, None]
        return f, nodes, ok, torch.where(ok, U[j[:, None], nodes], INF)

    a, b = torch.where(i >= 1, i - 1, i + 1), torch.where(i <= M - 2, i + 1, i - 1)
    f, node, ok, u = cands(i)
    phi = torch.zeros((G, 64, 8), dtype=torch.float64, device="cuda")
    phi[:, :, 0] = (st[node] - f[:, None]) / 4
    for col, j in ((1, a), (3, b)):
        _, nj, okj, uj = cands(j)
        q = nj.gather(1, uj.argmin(1, keepdim=True))[:, 0]
        there = okj.any(1)[:, None]
        d = sx[node] - sx[q][:, None]
        e = (mx[i] - mx[j])[:, None]
        phi[:, :, col:col + 2] = torch.where(there[:, :, None], (d - e) / 64, 0.0)
        if col == 1:
            phi[:, :, 5] = torch.where(there, torch.log((d.norm(dim=2) + 1) / (e.norm(dim=2) + 1)), 0.0)
    phi[:, :, 6] = u - u.amin(1, keepdim=True)
    phi[:, :, 7] = (i / (M - 1))[:, None]
    x = torch.cat([(DIM * m.desc.double())[i][:, None].expand(G, 64, DIM), DIM * s.desc.double()[node], phi], 2)
    x = torch.where(ok[:, :, None], x, 0.0).reshape(G * 64, -1)
    theta = torch.from_numpy(synth.pruner_init(DIM, seed % 1000).astype(np.float64)).cuda()
    sizes = [128 * (2 * DIM + 8), 128, 128 * 128, 128, 128, 1]
    W1, b1, W2, b2, w3, b3 = torch.split(theta, sizes)
    W1, W2 = W1.reshape(128, -1), W2.reshape(128, 128)
    h1 = (x @ W1.T + b1).relu_()
    h2 = (h1 @ W2.T + b2).relu_()
    sc = torch.where(ok, (h2 @ w3 + b3).reshape(G, 64), -INF)
    lab = torch.from_numpy(labels.astype(np.int64)).cuda()
    hit = (ok & (node == lab[:, None])).double()
    loss = (torch.logsumexp(sc, 1) - (torch.where(ok, sc, 0.0) * hit).sum(1)).mean()
    ds = ((torch.softmax(sc, 1) - hit) / G).reshape(-1)
    dz2 = ds[:, None] * w3 * (h2 > 0)
    dz1 = (dz2 @ W2) * (h1 > 0)
    grad = torch.cat([(dz1.T @ x).reshape(-1), dz1.sum(0), (dz2.T @ h1).reshape(-1), dz2.sum(0), ds @ h2,
                      ds.sum()[None]])
    return dict(loss=loss[None], grad=grad, scores=sc)


def exact(case, seed):
    c, k = case, case["kind"]
    models, scenes, sal = _inputs(c, seed)
    if k == "grad":
        return _exact_grad(c, models[0], scenes[0], seed)
    if k == "pruned":
        return None  # the kept lists are a ranking of 16-bit scores: no value of their own in 64 bits
    names = ("energy32", "energy64", "energy_u64")
    if k == "trellis":
        if c["T"] <= 0 and c["models"] * c["points"] ** 3 > 2e9:
            return None  # minutes
        rows = [_solve_trellis(m, scenes[0], c["T"]) for m in models]
        return dict(zip(names, (torch.stack([r[q] for r in rows]) for q in range(3))))
    if k == "match":
        m, s = models[0], scenes[0]
        cand, count = _window_cands(m, s, c["W"], c["K"], False, 0, s.n_frames - int(m.t[-1]))
        return dict(zip(names, _solve(m, s, cand, count, c["T"], c["dummy"], c["reading"], c["unary"] == "bf16")))
    if k == "chains":
        m, s = models[0], scenes[0]
        n = s.n_frames - int(m.t[-1])
        chains = [[] for _ in range(c["n_chains"])]
        for f in np.unique(m.t):
            at = np.flatnonzero(m.t == f)
            for q, p in enumerate(at[np.argsort(-sal[at], kind="stable")]):
                chains[q].append(p)
        rows = []
        for ch in (x for x in chains if len(x) >= 3):
            sub = _Set(m.xy[ch], m.t[ch], m.desc[torch.tensor(ch, device="cuda")])
            cand, count = _window_cands(sub, s, c["W"], c["K"], False, int(sub.t[0] - m.t[0]), n)
            rows.append(torch.stack(_solve(sub, s, cand, count, 10)))
        return dict(zip(names, torch.stack(rows).mean(0)))
    if work(c)["flops"] > 3e11:
        return None  # a whole batch takes minutes in 64 bits
    rows = []
    if k == "blocks":
        s = scenes[0]
        n, b = _n_blocks(c, models, s), c["block"]
        if len(models) * n * c["M"] * b ** 3 > 4e10:
            return None
        nodes = torch.arange(b, device="cuda") + torch.arange(n, device="cuda")[:, None]
        for m in models:
            have = s.n_frames - int(m.t[-1])
            cand = nodes[:, None].expand(n, c["M"], b).contiguous()
            got = torch.full((3, have), float("inf"), dtype=torch.float64, device="cuda")
            got[:, :n] = torch.stack(_solve(m, s, cand, torch.full((n, c["M"]), b, device="cuda"), c["T"]))
            rows.append(got)
    else:
        for m in models:
            for s in scenes:
                cand, count = _window_cands(m, s, c["W"], c["K"], c["density"], 0, s.n_frames - int(m.t[-1]))
                rows.append(torch.stack(_solve(m, s, cand, count, 10)))
    return dict(zip(names, torch.cat(rows, 1)))
