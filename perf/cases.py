"""The work that a program has this framework do, as cases that can be timed.

Rollouts of whole populations through ``Simulator`` (a pass is the rollout
and the fitness, state and counters on the device, as an evolutionary loop
reads them), and the steps of the learned pre-screen through ``Surrogate``:
features, prediction, one training epoch, top-k selection.  Inputs come from
the generators of ``workloads``, at the sizes of the benchmark, the tests and
the evolutionary loop, and ragged ones between.
"""
import ctypes
import math

import numpy as np
import torch

from paper_2502_11129_amd import sim as S
from paper_2502_11129_amd import surrogate as SU
from paper_2502_11129_amd import workloads as W

# The launch options that the autotuner chooses for random trees (bench.py);
# a program that tunes once keeps them for its run.
TUNED_TREES = dict(min_body_slots=32, slots32_min_nvc=24, min_nv_capacity=16, ncr_by_nvc={16: 8, 20: 4})


def listed():
    return [
        # a handful of robots: the simulator's latency (the smallest population of the tests)
        dict(name="snakes_16", kind="snakes", n=16, steps=1000),
        # free boxes dropped on a plane, no joints: the paper's BOX scene, whole horizon
        dict(name="boxes_4096", kind="boxes", n=4096, steps=2000),
        # the benchmark's population of uneven robots with tuned launch options
        dict(name="trees_8192_tuned", kind="trees", n=8192, steps=1000, tuned=True),
        # one generation's evaluation in the evolutionary loop, options left alone
        dict(name="trees_4096", kind="trees", n=4096, steps=1000, tuned=False),
        # the large uniform robots of the long-horizon and split runs
        dict(name="quadrupeds_8192", kind="quadrupeds", n=8192, steps=500),
        # the paper's BOX_AND_BALL scene, a size of its sweep
        dict(name="box_and_ball_32768", kind="box_and_ball", n=32768, steps=1000),
        # body-body contacts, a ragged population
        dict(name="quadrupeds_self_3001", kind="quadrupeds_self", n=3001, steps=500),
        # features of a labelled training set
        dict(name="features_200000", kind="features", n=200000),
        # predictions of a whole screening pool
        dict(name="predict_1000000", kind="predict", n=1000000),
        # predictions of a holdout of ragged size: one short chunk
        dict(name="predict_10007", kind="predict", n=10007),
        # one epoch over the evolutionary loop's pre-training set (six batches, the last one short)
        dict(name="train_24096", kind="train", n=24096, batch=4096),
        # the best 5 % of a screening pool
        dict(name="topk_1000003", kind="topk", n=1000003, k=50000),
    ]


# per kind: the range of population sizes and of steps (rollouts)
_ROLLOUTS = dict(snakes=((1, 2048), (100, 1000)), boxes=((64, 4096), (250, 2000)), trees=((64, 8192), (200, 1000)),
                 quadrupeds=((16, 8192), (100, 500)), box_and_ball=((32, 32768), (200, 1000)),
                 quadrupeds_self=((16, 3001), (100, 500)))
_SCREEN = dict(features=(500, 400000), predict=(1, 1000000), train=(300, 24096), topk=(1000, 1000003))


def _log_int(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    kind = rng.choice(sorted(_ROLLOUTS) + sorted(_SCREEN))
    if kind in _ROLLOUTS:
        (n0, n1), (t0, t1) = _ROLLOUTS[kind]
        c = dict(kind=kind, n=_log_int(rng, n0, n1), steps=_log_int(rng, t0, t1))
        if kind == "trees":
            c["tuned"] = rng.random() < 0.5
        return c
    c = dict(kind=kind, n=_log_int(rng, *_SCREEN[kind]))
    if kind == "train":
        c["batch"] = rng.choice([4096, 2048, 1000, 512])
    if kind == "topk":
        c["k"] = _log_int(rng, 1, c["n"] // 2)
    return c


# ----------------------------------------------------------------------------- inputs
def _population(case, seed):
    kind, n = case["kind"], case["n"]
    first = (seed % 1000003) * 40000  # the generators draw robot i from its own index
    if kind == "snakes":
        return W.snake(n, first=first)
    if kind == "boxes":
        return W.boxes(n, first=first)
    if kind == "trees":
        # the same bodies with other controllers, as when controllers are tuned
        g = W.random_genotypes(n, key=500)
        u = np.random.default_rng([20, seed]).random(g.cpg.shape)
        live = np.arange(20)[None, :, None] < g.nh[:, None, None]
        g.cpg = np.where(live, np.array([0.0, 1.0, 0.0]) + np.array([1.0, 5.0, 2.0 * math.pi]) * u, 0.0).astype(np.float32)
        return W.population_from_genotypes(g)
    if kind == "box_and_ball":
        return W.box_and_ball(n, first=first)
    pop = W.quadrupeds(n, first=first)
    pop.self_collision = kind == "quadrupeds_self"
    return pop


def _genotypes(n, seed, device):
    """n candidates: bodies of up to 8192 drawn ones in turn, every controller its own."""
    base = SU.W.genotype_arrays(W.random_genotypes(min(n, 8192), key=seed))
    at = torch.arange(n, device=device) % min(n, 8192)
    g = {k: torch.from_numpy(v).to(device)[at].contiguous() for k, v in base.items()}
    gen = torch.Generator(device=device).manual_seed(seed)
    u = torch.rand((n, 20, 3), generator=gen, device=device)
    lo = torch.tensor([0.0, 1.0, 0.0], device=device)
    width = torch.tensor([1.0, 5.0, 2.0 * math.pi], device=device)
    live = torch.arange(20, device=device)[None, :] < g["nh"][:, None]
    g["cpg"] = torch.where(live[:, :, None], lo + width * u, torch.zeros_like(u)).contiguous()
    return g


def _training_state(seed):
    """A network in mid-training: parameters, first and second moments, step count."""
    rng = np.random.default_rng([21, seed])
    p = W.mlp_init(seed)
    m = rng.normal(0.0, 1e-4, p.shape).astype(np.float32)
    v = (rng.uniform(0.5, 2.0, p.shape) * 1e-7).astype(np.float32)
    return p, m, v, 100


def _training_data(case, seed, device):
    """Targets of the n rows and the epoch's order."""
    rng = np.random.default_rng([22, seed])
    y = rng.normal(0.0, 1.0, case["n"]).astype(np.float32)
    perm = rng.permutation(case["n"]).astype(np.int32)
    return torch.from_numpy(y).to(device), torch.from_numpy(perm).to(device)


def _scores(n, seed, device):
    gen = torch.Generator(device=device).manual_seed(seed)
    return torch.randn(n, generator=gen, device=device)


def prepare(case, seed):
    device = torch.device("cuda")
    kind = case["kind"]
    st = dict(case)
    if kind in _ROLLOUTS:
        st["sim"] = S.Simulator(_population(case, seed), device=device, **(TUNED_TREES if case.get("tuned") else {}))
        return st
    if kind == "topk":
        st["sur"] = SU.Surrogate(seed=0, device=device)
        st["scores"] = _scores(case["n"], seed, device)
        return st
    st["sur"] = SU.Surrogate(seed=seed, device=device, max_batch=max(4096, case.get("batch", 0)))
    st["geno"] = _genotypes(case["n"], seed, device)
    if kind == "features":
        return st
    st["X"] = st["sur"].features(st.pop("geno"))
    if kind == "train":
        p, m, v, t = _training_state(seed)
        st["sur"].set_state(p, m, v, t)
        st["y"], st["perm"] = _training_data(case, seed, device)
        st["grad"] = torch.empty(SU.SUR_N_PARAMS, dtype=torch.float32, device=device)
    return st


def run(st):
    kind = st["kind"]
    if kind in _ROLLOUTS:
        sim = st["sim"]
        sim.rollout(st["steps"])
        fit = sim.fitness_device()
        q, v, k = sim.get_state_device()
        contact, clamp, status = sim.counters_device()
        return dict(fitness=fit, q=q, v=v, k=k, rows_contact=contact, rows_clamp=clamp, status=status)
    sur = st["sur"]
    if kind == "features":
        return sur.features(st["geno"])
    if kind == "predict":
        return sur.predict(st["X"])
    if kind == "topk":
        return sur.topk(st["scores"], st["k"])
    losses = sur.train_epoch(st["X"], st["y"], st["perm"], st["batch"])
    sur._check(sur.lib.sur_get_grad(sur.h, ctypes.c_void_p(st["grad"].data_ptr()), 1, sur.stream()))
    return dict(losses=losses, grad=st["grad"])


# ----------------------------------------------------------------------------- work
_N_WEIGHTS = 128 * 256 + 2 * 256 * 256 + 256  # products of one row's forward pass

# (hinges, bodies, sum of body depths, active contacts a step) of an average robot
_ROBOT = dict(snakes=(3, 4, 6, 4), boxes=(0, 1, 0, 4), trees=(12, 13, 26, 4), quadrupeds=(20, 21, 60, 5),
              box_and_ball=(0, 1, 0, 3.5), quadrupeds_self=(20, 21, 60, 5))


def work(case):
    kind, n = case["kind"], case["n"]
    if kind in _ROLLOUTS:
        nh, nb, depth, nc = _ROBOT[kind]
        ball = kind == "box_and_ball"
        nv = 6 + nh + (6 if ball else 0)
        step = 156 * nh + 594 * nb + 60 * depth + 72 * nh + (2 / 3) * nv ** 3 + 2 * nv ** 2 + 100
        step += nc * (50 + 9 * depth / nb + 6 * nv ** 2 + 6 * nv + 12 * 8 * nv)
        step += 130 if ball else 0
        step += 6 * nb * (nb - 1) if kind == "quadrupeds_self" else 0
        nq = nv + (2 if ball else 1)
        return dict(bytes=n * (4 * (24 * nb + 16) + 12 * (nq + nv) + 32), flops=n * case["steps"] * step)
    if kind == "features":
        return dict(bytes=n * (4 + 60 + 240 + 256), flops=n * 200)
    if kind == "predict":
        return dict(bytes=n * (256 + 4), flops=2 * n * _N_WEIGHTS)
    if kind == "topk":
        return dict(bytes=4 * n + 4 * case["k"], flops=n)
    batches = -(-n // case["batch"])
    flops = 2 * n * (2 * _N_WEIGHTS + 2 * 256 * 256) + 12 * batches * SU.SUR_N_PARAMS
    return dict(bytes=n * (256 + 8) + batches * 6 * 4 * SU.SUR_N_PARAMS, flops=flops)


# ----------------------------------------------------------------------------- 64-bit results
def _exact_features(case, seed):
    g = {k: v.cpu().numpy() for k, v in _genotypes(case["n"], seed, torch.device("cuda")).items()}
    n, nh = case["n"], g["nh"].astype(np.int64)
    rows = np.arange(n)
    live = np.arange(20)[None, :] < nh[:, None]
    par, face, axis = (g[k].astype(np.int64) for k in ("parent", "face", "axis"))
    depth = np.zeros((n, 21), np.int64)
    limb = np.zeros((n, 21), np.int64)
    size = np.zeros((n, 21), np.int64)
    for j in range(20):
        p = np.where(live[:, j], par[:, j], 0)
        depth[:, j + 1] = np.where(live[:, j], depth[rows, p] + 1, 0)
        limb[:, j + 1] = np.where(live[:, j], np.where(p == 0, j + 1, limb[rows, p]), 0)
        np.add.at(size, (rows[live[:, j]], limb[live[:, j], j + 1]), 1)
    F = np.zeros((n, 128))
    cpg = g["cpg"].astype(np.float64)
    F[:, 0:20] = np.where(live, cpg[:, :, 0], 0.0)
    F[:, 20:40] = np.where(live, cpg[:, :, 1] / 6.0, 0.0)
    F[:, 40:60] = np.where(live, cpg[:, :, 2] / (2 * math.pi), 0.0)
    F[:, 60:80] = np.where(live, np.where(axis == 0, 1.0, -1.0), 0.0)
    F[:, 80:100] = depth[:, 1:] / 4.0
    nz = (live & (axis == 0)).sum(1)
    F[:, 100], F[:, 101], F[:, 102], F[:, 103] = nh / 20.0, nz / 20.0, (nh - nz) / 20.0, depth.max(1) / 4.0
    for d in range(1, 6):
        F[:, 103 + d] = (depth[:, 1:] == d).sum(1) / 20.0
    root = live & (par == 0)
    lo, hi = (1, 2, 3, 5, 9), (1, 2, 4, 8, 99)
    for b in range(5):
        F[:, 109 + b] = 0.25 * (root & (size[:, 1:] >= lo[b]) & (size[:, 1:] <= hi[b])).sum(1)
    for f in range(4):
        F[:, 114 + f] = (root & (face == f)).any(1)
    return torch.from_numpy(F)


def _layers(p):
    """Weights (as the products read them, in BF16) and biases of a flat parameter vector, in 64 bits."""
    out, at = [], 0
    for i, o in ((128, 256), (256, 256), (256, 256), (256, 1)):
        w = p[at:at + i * o].reshape(i, o)
        out.append((w.float().to(torch.bfloat16).double(), p[at + i * o:at + i * o + o]))
        at += i * o + o
    return out


def _phi(z):
    return 0.5 * (1.0 + torch.erf(z / math.sqrt(2.0)))


def _exact_predict(case, seed):
    device = torch.device("cuda")
    X = _exact_features(case, seed).to(device).to(torch.bfloat16)
    layers = _layers(torch.from_numpy(W.mlp_init(seed)).to(device).double())
    out = []
    for r in range(0, case["n"], 65536):
        h = X[r:r + 65536].double()
        for w, b in layers[:3]:
            z = h @ w + b
            h = z * _phi(z)
        out.append((h @ layers[3][0] + layers[3][1])[:, 0])
    return torch.cat(out)


def _exact_train(case, seed):
    device = torch.device("cuda")
    X = _exact_features(case, seed).to(device).to(torch.bfloat16)
    y, perm = _training_data(case, seed, device)
    p, m, v, t = _training_state(seed)
    p, m, v = (torch.from_numpy(a).to(device).double() for a in (p, m, v))
    losses, grad = [], None
    for r in range(0, case["n"], case["batch"]):
        idx = perm[r:r + case["batch"]].long()
        layers, hs, zs = _layers(p), [X[idx].double()], []
        for w, b in layers[:3]:
            zs.append(hs[-1] @ w + b)
            hs.append(zs[-1] * _phi(zs[-1]))
        res = (hs[3] @ layers[3][0] + layers[3][1])[:, 0] - y[idx].double()
        losses.append((res * res).mean())
        d = (2.0 / len(idx) * res)[:, None]
        parts = []
        for l in (3, 2, 1, 0):
            parts = [(hs[l].T @ d).reshape(-1), d.sum(0)] + parts
            if l:
                z = zs[l - 1]
                d = (d @ layers[l][0].T) * (_phi(z) + z * torch.exp(-0.5 * z * z) / math.sqrt(2.0 * math.pi))
        grad = torch.cat(parts)
        t += 1
        m, v = 0.9 * m + 0.1 * grad, 0.999 * v + 0.001 * grad * grad
        p = p - 1e-3 * (m / (1 - 0.9 ** t)) / ((v / (1 - 0.999 ** t)).sqrt() + 1e-8)
    return dict(losses=torch.stack(losses), grad=grad)


def exact(case, seed):
    """64-bit results of the pre-screen's steps.  None for a rollout (hundreds of
    steps of an articulated robot take minutes in plain array code) and for
    top-k, whose outputs are whole numbers."""
    if case["kind"] == "features":
        return _exact_features(case, seed)
    if case["kind"] == "predict":
        return _exact_predict(case, seed)
    if case["kind"] == "train":
        return _exact_train(case, seed)
    return None
