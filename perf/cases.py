"""Performance cases of the prefix-placement planner.

Each case is one call that a user of this library makes, through its public
binding, on seeded synthetic inputs of the shapes the planner serves:

  plan / plan_f64        the whole planner on device-resident inputs with a
                         reusable context (integer or real-valued costs)
  plan_host              the same on host arrays, copies included
  replan / replan_f64    epoch re-planning on host arrays
  rooted_dp(_f64)        one exact rooted-tree solve on host arrays
  marginal               one worker's exact marginals on host arrays
  objective              the allocation-free objective on device arrays

Trees: "gw" Galton-Watson, "rag" shared prompt -> templates -> documents,
"chat" conversation chains on a Galton-Watson base, "deep" one long
regenerated conversation, "forest" a random forest with shuffled ids.
"""

import math

import numpy as np
import torch

from paper_2608_01655_amd import binding as B
from paper_2608_01655_amd import workloads as W


def _case(name, kind, tree, n, m, k, starts=8, rounds=0, fetch="pair", horizon=0, k_hi=0,
          safeguards=False):
    """k: chunks per worker; k_hi > 0: drawn per worker from [k, k_hi]."""
    c = dict(kind=kind, tree=tree, n=n, m=m, k=k, k_hi=k_hi, starts=starts, rounds=rounds,
             fetch=fetch, horizon=horizon, safeguards=safeguards)
    if name is not None:
        c["name"] = name
    return c


def listed():
    return [
        # the smallest plan: a two-worker pool with requester-side costs,
        # where launches and host work are all there is
        _case("plan_host_tiny", "plan_host", "gw", 200, 2, 40, starts=1, rounds=3,
              fetch="requester"),
        # a small pool re-planned between epochs with the comparators asked
        # for (six workers, 10% budgets, the size of one document benchmark)
        _case("replan_f64_small", "replan_f64", "rag", 183, 6, 18, starts=8, fetch="requester",
              horizon=1000, safeguards=True),
        # a small shared tree, four workers
        _case("plan_tree2k", "plan", "gw", 2_000, 4, 256, starts=4),
        # the RAG-shaped pool
        _case("plan_rag10k", "plan", "rag", 10_000, 8, 1_024, starts=8),
        # the bench's default: a deployment-sized pool
        _case("plan_tree50k", "plan", "gw", 50_000, 16, 4_096, starts=8),
        # multi-turn conversations, uneven workers, many starts: the largest
        _case("plan_chat50k", "plan", "chat", 50_000, 16, 2_048, starts=32, k_hi=8_192),
        # real-valued costs at the size the method's solver time is quoted on
        _case("plan_f64_tree50k_k128", "plan_f64", "gw", 50_000, 16, 128, starts=8),
        # and its n = 10,000, M = 4 point: every order as a start
        _case("plan_f64_rag10k_m4", "plan_f64", "rag", 10_000, 4, 128, starts=0),
        # an epoch's re-plan through host arrays, odd sizes
        _case("replan_rag9973", "replan", "rag", 9_973, 6, 997, starts=8, horizon=1000),
        # one exact tree solve: shuffled ids, odd sizes
        _case("rooted_dp_20011", "rooted_dp", "forest", 20_011, 1, 1_531),
        # one exact tree solve on a long regenerated conversation
        _case("rooted_dp_f64_deep", "rooted_dp_f64", "deep", 6_001, 1, 500),
        # a serving loop's evaluation of its current placement
        _case("objective_rag10k", "objective", "rag", 10_000, 8, 1_024),
    ]


def draw(rng):
    def log_int(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    kind = rng.choice(["plan", "plan", "plan", "plan_f64", "plan_f64", "plan_host", "replan",
                       "replan_f64", "rooted_dp", "rooted_dp_f64", "marginal", "objective"])
    fetch = rng.choice(["pair", "pair", "requester"])
    if kind in ("rooted_dp", "rooted_dp_f64"):
        tree = rng.choice(["forest", "gw", "rag", "deep"])
        n = log_int(150, 6_500 if tree == "deep" else 50_000)
        return _case(None, kind, tree, n, 1, max(1, int(n * rng.uniform(0.01, 0.12))))
    if kind in ("marginal", "objective"):
        return _case(None, kind, rng.choice(["gw", "rag"]), log_int(200, 50_000),
                     rng.randint(1, 16), 64, fetch=fetch)
    small = kind in ("plan_host", "replan", "replan_f64")
    n = log_int(150, 20_000 if small else 50_000)
    m = rng.randint(2, 16)
    k = max(4, int(n * math.exp(rng.uniform(math.log(0.003), math.log(0.15)))))
    k = min(k, 8_000)
    tree = rng.choice(["gw", "rag", "chat"]) if n >= 2_000 else rng.choice(["gw", "rag"])
    starts = rng.choice([1, 2, 4, 8, 8, 16])
    if m <= 4 and rng.random() < 0.3:
        starts = 0
    return _case(None, kind, tree, n, m, k, starts=starts, rounds=rng.choice([0, 0, 0, 2]),
                 fetch=fetch, horizon=rng.choice([1, 100, 1000]),
                 k_hi=rng.choice([0, 0, min(2 * k, 8_192)]), safeguards=rng.random() < 0.25)


# ------------------------------------------------------------ inputs ----

def _tree(case, rng):
    n = case["n"]
    if case["tree"] == "forest":
        return W.random_forest(n, rng)
    if case["tree"] == "deep":
        return W.regenerated_conversation(n, rng)
    if case["tree"] == "gw":
        par = W.galton_watson_tree(n, 2.2, 16, rng)
    elif case["tree"] == "rag":
        par = W.rag_tree(n, min(40, max(2, n // 25)), rng)
    else:
        par = W.chain_tree(n, (7 * n) // 10, 2.2, 16, 64, rng)
    parent, _ = W._relabel_preorder(par)
    return parent


def _tree_profit(parent, rng):
    """Profits of one solve: integer demand that grows towards the roots
    (Zipf over the nodes, summed over each subtree along depth order) times
    a recompute cost per chunk."""
    n = parent.shape[0]
    own = np.floor(10 ** 6 / (rng.permutation(n) + 1.0)).astype(np.int64)
    depth = np.full(n, -1, np.int64)
    for v in range(n):
        path = []
        u = v
        while u >= 0 and depth[u] < 0:
            path.append(u)
            u = parent[u]
        d = -1 if u < 0 else int(depth[u])
        for x in reversed(path):
            d += 1
            depth[x] = d
    lam = own.copy()
    for v in np.argsort(-depth, kind="stable"):
        p = parent[v]
        if p >= 0:
            lam[p] += lam[v]
    # the demand that reaches a node is held down where chains are long
    lam = np.minimum(lam, 10 ** 8)
    return lam * (W.COST_A_US + W.COST_B_US * np.minimum(depth, 64))


def _inputs(case, seed):
    rng = np.random.default_rng(seed)
    parent = _tree(case, rng)
    n, m = case["n"], case["m"]
    assert parent.shape[0] == n
    if case["kind"].startswith("rooted_dp"):
        p = _tree_profit(parent, rng)
        if case["kind"] == "rooted_dp_f64":
            p = p / 1000.0 * rng.uniform(0.75, 1.25, size=n)
        return dict(parent=parent, profit=p, k=case["k"])
    depth = W._depths(parent)
    zipf = {"gw": 1.0, "rag": 0.9, "chat": 1.2}[case["tree"]]
    lam = W.zipf_leaf_demand(parent, m, zipf, 2_000 * n, rng)
    w = W.depth_linear_recompute(depth, W.H10_CYCLE[(np.arange(m) + 1) % 3])
    if case["fetch"] == "requester":
        f = W.requester_fetch(m, n, 100_700)
    else:
        f = W.pairwise_fetch(m, n, 1.0, 25.0, rng)
    if case["k_hi"] > 0:
        cap = rng.integers(case["k"], case["k_hi"] + 1, size=m).astype(np.int32)
    else:
        cap = np.full(m, case["k"], np.int32)
    x = dict(parent=parent, lam=lam, w=w, f=f, cap=cap, order_seed=int(seed) % 1000)
    if case["kind"].startswith("replan"):
        x["lam"] = W.shift_routing(parent, lam, 1, 2)
        x["incumbent"] = W.prefix_incumbent(n, cap)
    if case["kind"] in ("marginal", "objective"):
        x["target"] = W.prefix_incumbent(n, cap)
        x["h"] = int(rng.integers(0, m))
    if case["kind"].endswith("f64"):
        lo, hi = 0.75, 1.25
        x["lam"] = x["lam"] * rng.uniform(lo, hi, size=lam.shape)
        x["w"] = w / 1000.0 * rng.uniform(lo, hi, size=w.shape)
        # one factor per requester and chunk, so that requester-side costs
        # stay requester-side
        x["f"] = f / 1000.0 * rng.uniform(lo, hi, size=(1, m, n))
        x["eps"] = 1e-9 * float((x["lam"] * x["w"]).sum())
    return x


def prepare(case, seed):
    x = _inputs(case, seed)
    x["case"] = case
    kind = case["kind"]
    x["opts"] = dict(n_starts=case["starts"], max_rounds=case["rounds"],
                     order_seed=x.get("order_seed", 0),
                     flags=B.PP_F_SAFEGUARDS if case["safeguards"] else 0)
    if kind in ("plan", "plan_f64", "objective"):
        dev = torch.device("cuda", torch.cuda.current_device())
        for key in ("lam", "w", "f"):
            x[key] = torch.from_numpy(np.ascontiguousarray(x[key])).to(dev)
        if kind == "objective":
            x["target"] = torch.from_numpy(x["target"]).to(dev)
        else:
            x["target"] = torch.zeros((case["m"], case["n"]), dtype=torch.uint8, device=dev)
            x["ctx"] = B.Context(dev.index)
        torch.cuda.synchronize()
    return x


def _plan_outputs(p):
    return dict(target=p.target, objective=p.objective, best_start=p.best_start,
                updates=p.updates, dp_cells=p.dp_cells, start_objective=p.start_objective,
                start_sweeps=p.start_sweeps, start_accepts=p.start_accepts,
                standalone=p.standalone, orders=p.orders,
                safeguards_run=int(p.safeguards_run),
                safeguard_objective=list(p.safeguard_objective))


def run(state):
    s = state
    kind = s["case"]["kind"]
    if kind == "plan":
        return _plan_outputs(s["ctx"].pp_plan_device(
            s["parent"], s["lam"], s["w"], s["f"], s["cap"], s["target"], **s["opts"]))
    if kind == "plan_f64":
        return _plan_outputs(s["ctx"].pp_plan_f64_device(
            s["parent"], s["lam"], s["w"], s["f"], s["cap"], s["target"], epsilon=s["eps"],
            **s["opts"]))
    if kind == "plan_host":
        return _plan_outputs(B.pp_plan(s["parent"], s["lam"], s["w"], s["f"], s["cap"],
                                       **s["opts"]))
    if kind in ("replan", "replan_f64"):
        args = (s["parent"], s["lam"], s["w"], s["f"], s["cap"], s["incumbent"],
                s["case"]["horizon"])
        if kind == "replan":
            r = B.pp_replan(*args, **s["opts"])
        else:
            r = B.pp_replan_f64(*args, epsilon=s["eps"], **s["opts"])
        return dict(target=r.target, adopt=int(r.adopt),
                    incumbent_objective=r.incumbent_objective,
                    materialization_cost=r.materialization_cost, plan=_plan_outputs(r.plan))
    if kind == "rooted_dp":
        return B.pp_rooted_dp(s["parent"], s["profit"], s["k"])
    if kind == "rooted_dp_f64":
        return B.pp_rooted_dp_f64(s["parent"], s["profit"], s["k"])
    if kind == "marginal":
        return B.pp_marginal(s["lam"], s["w"], s["f"], s["target"], s["h"])
    return B.pp_objective_device_noalloc(s["lam"], s["w"], s["f"], s["target"])


def _starts(case):
    if case["starts"] > 0:
        return case["starts"]
    return math.factorial(case["m"]) if case["m"] <= 5 else 8


def work(case):
    """Inputs once, outputs once.  A plan evaluates every worker's marginals
    (about four operations per requester and chunk) for the standalone
    scores, the greedy pass and at least the one sweep that accepts nothing;
    the tree solves are counted as one comparison per chunk, since no one
    table of them is needed."""
    n, m, kind = case["n"], case["m"], case["kind"]
    if kind.startswith("rooted_dp"):
        return {"bytes": n * (4 + 8 + 1) + 8, "flops": n}
    inputs = 8 * (2 * m * n + m * (m - 1) * n)
    if kind in ("marginal", "objective"):
        out = 8 * n + 8 if kind == "marginal" else 8
        return {"bytes": inputs + m * n + out, "flops": 4 * m * m * n}
    updates = m + 2 * _starts(case) * m
    extra = 2 * m * n if kind.startswith("replan") else 0
    return {"bytes": inputs + 4 * n + m * n + extra, "flops": updates * (4 * m + 1) * n}


def tolerance(case):
    """Every result is pinned bit for bit: integer sums, a fixed order of
    rounding in the real-valued tree solve, exact sums of the rounded terms
    for real-valued objectives, and deterministic ties."""
    return "exact"


# ------------------------------------------- the same in plain numpy ----

def _preorder(parent):
    n = len(parent)
    kids = [[] for _ in range(n)]
    roots = []
    for v in range(n):
        (kids[parent[v]] if parent[v] >= 0 else roots).append(v)
    order, stack = [], list(reversed(roots))
    while stack:
        v = stack.pop()
        order.append(v)
        stack.extend(reversed(kids[v]))
    pos = np.empty(n, np.int64)
    pos[order] = np.arange(n)
    size = np.ones(n, np.int64)
    for q in range(n - 1, -1, -1):
        p = parent[order[q]]
        if p >= 0:
            size[pos[p]] += size[q]
    return np.array(order), np.arange(n) + size


def _solve(nxt, p, k):
    """Rooted-tree knapsack in preorder: D[i][j] = max(D[next(i)][j],
    p_i + D[i+1][j-1]), a node taken only if strictly better."""
    n = len(p)
    k = min(int(k), n)
    sel = np.zeros(n, np.uint8)
    if k == 0:
        return sel, p.dtype.type(0)
    uses = np.zeros(n + 1, np.int64)
    for q in range(n):
        uses[nxt[q]] += 1
    rows = {n: np.zeros(k + 1, p.dtype)}
    below = rows[n]
    choice = np.zeros((n, (k + 7) // 8), np.uint8)
    for q in range(n - 1, -1, -1):
        sk = rows[nxt[q]]
        t = p[q] + below[:-1]
        take = t > sk[1:]
        choice[q] = np.packbits(take)
        row = sk.copy()
        np.copyto(row[1:], t, where=take)
        uses[nxt[q]] -= 1
        if uses[nxt[q]] == 0:
            del rows[nxt[q]]
        if uses[q]:
            rows[q] = row
        below = row
    q, j = 0, k
    while q < n and j > 0:
        if (choice[q, (j - 1) >> 3] >> (7 - ((j - 1) & 7))) & 1:
            sel[q] = 1
            q += 1
            j -= 1
        else:
            q = int(nxt[q])
    return sel, below[k]


class _Planner:
    def __init__(self, x, f64):
        self.order, self.nxt = _preorder(x["parent"])
        o = self.order
        self.f64 = f64
        self.lam, self.w = x["lam"][:, o], x["w"][:, o]
        self.m, self.n = self.lam.shape
        self.q = np.maximum(self.w[None] - x["f"][:, :, o], 0)  # [holder][requester][b]
        for h in range(self.m):
            self.q[h, h] = self.w[h]
        self.f = x["f"][:, :, o]
        self.cap = [min(int(c), self.n) for c in x["cap"]]

    def best(self, T, without=-1):
        v = np.zeros((self.m, self.n), self.w.dtype)
        for h in range(self.m):
            if h != without:
                np.maximum(v, np.where(T[h][None] > 0, self.q[h], 0), out=v)
        return v

    def terms(self, T):
        return self.lam * self.best(T)

    def total(self, terms):
        return math.fsum(terms.ravel()) if self.f64 else int(terms.sum())

    def better(self, a, b, eps):
        """sum(a) > sum(b) + eps, exactly."""
        if not self.f64:
            return int(a.sum()) > int(b.sum())
        keep = a != b
        return math.fsum(np.concatenate([a[keep], -b[keep], [-eps]])) > 0

    def marginal(self, T, h):
        v = self.best(T, h)
        p = np.zeros(self.n, self.w.dtype)
        for r in range(self.m):
            p = p + self.lam[r] * np.maximum(self.q[h, r] - v[r], 0)
        return p

    def caller(self, T):
        out = np.zeros_like(T)
        out[:, self.order] = T
        return out


def _orders(m, starts, seed, score):
    if starts == 0 and m <= 5:
        import itertools
        return np.array(list(itertools.permutations(range(m))), np.int32)
    starts = starts or 8
    first = sorted(range(m), key=lambda h: -score[h])
    out = []
    for s in range(starts):
        if s == 0:
            out.append(first)
        elif s == 1:
            out.append(first[::-1])
        else:
            state, o = (seed + s) % 2 ** 64, list(range(m))
            for i in range(m - 1, 0, -1):
                state = (state + 0x9E3779B97F4A7C15) % 2 ** 64
                z = state
                z = ((z ^ (z >> 30)) * 0xBF58476D1CE4E5B9) % 2 ** 64
                z = ((z ^ (z >> 27)) * 0x94D049BB133111EB) % 2 ** 64
                z ^= z >> 31
                j = z % (i + 1)
                o[i], o[j] = o[j], o[i]
            out.append(o)
    return np.array(out, np.int32)


def _exact_plan(case, x, f64):
    P = _Planner(x, f64)
    m, n, eps = P.m, P.n, x.get("eps", 0)
    dt = np.float64 if f64 else np.int64
    empty = np.zeros((m, n), np.uint8)
    score = np.array([_solve(P.nxt, P.marginal(empty, h), P.cap[h])[1] for h in range(m)], dt)
    orders = _orders(m, case["starts"], x["order_seed"], score)
    cells_pass = n * sum(P.cap)
    S = len(orders)
    sweeps, accepts, objs, placed = np.zeros(S, np.int32), np.zeros(S, np.int32), [], []
    updates, cells = m, cells_pass
    for s, order in enumerate(orders):
        T = empty.copy()
        for h in order:
            T[h] = _solve(P.nxt, P.marginal(T, h), P.cap[h])[0]
        cur = P.terms(T)
        while True:
            improved = False
            for h in order:
                T2 = T.copy()
                T2[h] = _solve(P.nxt, P.marginal(T, h), P.cap[h])[0]
                new = P.terms(T2)
                if P.better(new, cur, eps):
                    T, cur, improved = T2, new, True
                    accepts[s] += 1
            sweeps[s] += 1
            if not improved or (case["rounds"] and sweeps[s] >= case["rounds"]):
                break
        updates += m * (1 + int(sweeps[s]))
        cells += cells_pass * (1 + int(sweeps[s]))
        objs.append(cur)
        placed.append(T)
    best = 0
    for s in range(1, S):
        if P.better(objs[s], objs[best], 0):
            best = s
    win, win_terms, best_start = placed[best], objs[best], best
    sg_run, sg_obj = 0, [dt(0).item()] * 3
    if case["safeguards"] and (case["fetch"] == "requester" or m == 1):
        sg_run = 1
        updates += 3 * m
        cells += 3 * cells_pass
        cand = []
        for mode in range(3):
            T, union = empty.copy(), np.zeros(n, bool)
            for h in range(m):
                L, Wh = P.lam[h], P.w[h]
                if mode == 0 or (mode == 2 and m == 1):
                    p = L * Wh
                elif mode == 1:
                    p = L + np.zeros(n, dt)
                else:
                    F = P.f[1 if h == 0 else 0, h]
                    a = L * np.minimum(Wh, F)
                    p = np.where(union, a, a + L * np.maximum(Wh - F, 0))
                T[h] = _solve(P.nxt, p, P.cap[h])[0]
                union |= T[h] > 0
            cand.append((T, P.terms(T)))
        sg_obj = [P.total(t) for _, t in cand]
        for c, (T, t) in enumerate(cand):
            if P.better(t, win_terms, 0):
                win, win_terms, best_start = T, t, S + c
    out = dict(target=P.caller(win), objective=P.total(win_terms), best_start=best_start,
               updates=updates, dp_cells=cells,
               start_objective=np.array([P.total(t) for t in objs], dt), start_sweeps=sweeps,
               start_accepts=accepts, standalone=score, orders=orders, safeguards_run=sg_run,
               safeguard_objective=sg_obj)
    return out, P, win, win_terms


def exact(case, seed):
    n, m, kind = case["n"], case["m"], case["kind"]
    k = max(case["k"], case["k_hi"])
    row = 6e-6 + 4e-9 * min(k, n)  # seconds per row of one tree solve
    if not kind.startswith("rooted_dp") and kind not in ("marginal", "objective"):
        updates = m + _starts(case) * m * 6
        if updates * (n * row + m * m * n * 4e-9) > 18 or m * m * n > 4e7:
            return None
    x = _inputs(case, seed)
    f64 = kind.endswith("f64")
    if kind.startswith("rooted_dp"):
        order, nxt = _preorder(x["parent"])
        sel, val = _solve(nxt, x["profit"][order], x["k"])
        out = np.zeros(n, np.uint8)
        out[order] = sel
        return out, val.item()
    if kind in ("marginal", "objective"):
        x["parent"] = np.full(n, -1, np.int32)
        P = _Planner(x, False)
        if kind == "objective":
            return P.total(P.terms(x["target"]))
        v = P.best(x["target"], x["h"])
        return P.marginal(x["target"], x["h"]), int((P.lam * v).sum())
    out, P, win, win_terms = _exact_plan(case, x, f64)
    if not kind.startswith("replan"):
        return out
    inc = x["incumbent"][:, P.order]
    inc_terms = P.terms(inc)
    costs = []
    for r in range(m):
        c = P.w[r].copy()
        for h in range(m):
            if h != r:
                c = np.where(inc[h] > 0, np.minimum(c, P.f[h, r]), c)
        costs.append(c[(win[r] > 0) & (inc[r] == 0)])
    costs = np.concatenate(costs)
    cost = P.total(costs)
    if f64:
        gain = math.fsum(np.concatenate([win_terms.ravel(), -inc_terms.ravel()]))
    else:
        gain = P.total(win_terms) - P.total(inc_terms)
    adopt = int(case["horizon"] * gain > cost)
    return dict(target=P.caller(win) if adopt else x["incumbent"], adopt=adopt,
                incumbent_objective=P.total(inc_terms), materialization_cost=cost, plan=out)
