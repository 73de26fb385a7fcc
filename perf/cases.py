"""Performance cases: the calls a structure-learning program makes, over their real range.

A program builds the score table of its dataset, scores orders on it (one at a
time or in batches), runs Metropolis-Hastings chains (one dataset or many,
uniform or learned swaps) and trains the learned proposal's network.  The listed
cases take those steps at the sizes of the seeded workloads in
``paper_1210_5128_amd/datagen.py`` and of ``bench.py``; ``draw`` gives others of
the same ranges.  Datasets are complete discrete samples of random networks with
at most four parents per node; every size, arity and seed is in the case.
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_1210_5128_amd import bnos, datagen

N_MAX, SAMPLES_MAX = 60, 5000


# ------------------------------------------------------------------ cases

def listed():
    return [
        # an interactive caller scoring one order of a small network from host memory (`tiny8`)
        dict(name="order_host_8", kind="score", entry="host", n=8, N=200, arities="2", dmax=3, K=3, prior=False,
             orders=1, nodes=False),
        # the headline: one order per call on the 60-node mixed-arity table (`mixed60`), device buffers
        dict(name="order_60", kind="score", entry="device", n=60, N=5000, arities="234", dmax=4, K=4, prior=True,
             orders=1, nodes=False),
        # a serving loop that may not allocate: an odd batch with every per-node output (`mixed40`)
        dict(name="batch37_40", kind="score", entry="noalloc", n=40, N=2000, arities="234", dmax=4, K=4, prior=True,
             orders=37, nodes=True),
        # a population of orders scored in one call on the 60-node table
        dict(name="batch256_60", kind="score", entry="device", n=60, N=5000, arities="234", dmax=4, K=4, prior=True,
             orders=256, nodes=False),
        # the structure-recovery study's run: one chain, max-score target, a record of the best graphs (`roc20`)
        dict(name="chain1_20", kind="chains", n=20, N=1000, arities="2", dmax=3, K=4, prior=False, chains=1,
             iterations=1000, target=1, topk=8, learned=False, tables=1),
        # posterior sampling with many chains (`mixed40`)
        dict(name="chains256_40", kind="chains", n=40, N=2000, arities="234", dmax=4, K=4, prior=True, chains=256,
             iterations=128, target=0, topk=0, learned=False, tables=1),
        # posterior sampling on the largest workload (`mixed60`)
        dict(name="chains256_60", kind="chains", n=60, N=5000, arities="234", dmax=4, K=4, prior=True, chains=256,
             iterations=128, target=0, topk=0, learned=False, tables=1),
        # several datasets of uneven size advanced together (the `uneven` family)
        dict(name="multi8x32", kind="chains", n=60, N=5000, arities="234", dmax=3, K=4, prior=False, chains=32,
             iterations=64, target=0, topk=0, learned=False, tables=8),
        # chains driven by the learned swap proposal
        dict(name="learned64_40", kind="chains", n=40, N=2000, arities="234", dmax=4, K=4, prior=True, chains=64,
             iterations=128, target=0, topk=0, learned=True, tables=1),
        # a small dataset's table, read back whole (`prior20`)
        dict(name="build_20", kind="build", n=20, N=1000, arities="3", dmax=4, K=4, prior=True, orders=0),
        # the largest workload's table, and the first orders scored on it (`mixed60`)
        dict(name="build_60", kind="build", n=60, N=5000, arities="234", dmax=4, K=4, prior=True, orders=8),
        # training the learned proposal on harvested moves
        dict(name="train_60", kind="mlp", op="train", n=60, rows=8192, batch=1024, epochs=2),
    ]


def _log_int(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    """One more case of the ranges above."""
    kind = rng.choice(["score", "score", "chains", "chains", "build", "mlp"])
    if kind == "mlp":
        op = rng.choice(["forward", "grad", "train"])
        n = rng.randint(5, N_MAX)
        rows = _log_int(rng, 16, 8192)
        if op != "train":
            return dict(kind="mlp", op=op, n=n, rows=rows)
        return dict(kind="mlp", op=op, n=n, rows=rows, batch=min(rows, _log_int(rng, 64, 1024)), epochs=rng.randint(1, 2))
    n = _log_int(rng, 6, N_MAX)
    c = dict(kind=kind, n=n, N=_log_int(rng, 150, SAMPLES_MAX), arities=rng.choice(["2", "3", "23", "234"]),
             dmax=rng.randint(2, 4), prior=rng.random() < 0.5)
    # size limit 4 as in the workloads, smaller sets, and larger ones on small networks
    c["K"] = min(n - 1, rng.choice([2, 3, 4, 4, 4, 5] if n <= 24 else [2, 3, 4, 4, 4]))
    if kind == "score":
        c["entry"] = rng.choice(["device", "device", "noalloc", "host"])
        c["orders"] = 1 if c["entry"] == "host" else rng.choice([1, _log_int(rng, 2, 256)])
        c["nodes"] = c["entry"] != "host" and rng.random() < 0.5
    elif kind == "build":
        c["orders"] = rng.choice([0, 1, 8]) if n <= 24 else rng.choice([1, 8])
    else:
        c["learned"] = rng.random() < 0.25
        c["tables"] = 1 if c["learned"] else rng.choice([1, 1, 1, rng.randint(2, 6)])
        c["chains"] = _log_int(rng, 1, 64 if c["tables"] > 1 else 256)
        c["iterations"] = rng.randint(32, 128) if c["chains"] > 16 or c["tables"] > 1 else rng.randint(100, 600)
        c["target"] = rng.choice([0, 0, 1])
        c["topk"] = rng.choice([0, 0, 5])
    return c


# ------------------------------------------------------------------ inputs

def _dataset(case, seed, n=None, N=None):
    n = case["n"] if n is None else n
    N = case["N"] if N is None else N
    net = datagen.random_network(n, N, [int(a) for a in case["arities"]], min(case["dmax"], n - 1), seed)
    prior = datagen.random_prior(n, seed + 1) if case["prior"] else None
    return net, prior


def _dims(case):
    """(n, N) of each table: the case's, or uneven ones as in the uneven family (20..n nodes, N/5..N samples)."""
    if case.get("tables", 1) == 1:
        return [(case["n"], case["N"])]
    rng = np.random.default_rng([7, case["n"], case["N"], case["tables"]])
    lo = min(20, case["n"])
    return [(int(rng.integers(lo, case["n"] + 1)), int(rng.integers(max(1, case["N"] // 5), case["N"] + 1)))
            for _ in range(case["tables"])]


def _samples(case, seed):
    """Feature rows like a harvest's (position, local scores, prior sums, row statistics) and swapped pairs."""
    rng = np.random.default_rng([5, seed])
    R, n = case["rows"], case["n"]
    f = np.empty((R, n, 8), dtype=np.float32)
    stat = np.stack([rng.normal(0, 5, n), rng.normal(0, 5, n), rng.normal(-4000, 800, n), rng.normal(-4600, 800, n),
                     rng.uniform(50, 400, n)], axis=1)
    f[..., 0] = np.argsort(rng.random((R, n)), axis=1) / n
    f[..., 1] = stat[:, 2] - rng.exponential(60, (R, n))
    f[..., 2] = rng.exponential(8, (R, n))
    f[..., 3:] = stat.astype(np.float32)
    a = rng.integers(0, n, R)
    b = (a + rng.integers(1, n, R)) % n
    pairs = np.stack([a, b], axis=1).astype(np.int32)
    flat = f.reshape(-1, 8).astype(np.float64)
    mu, sd = flat.mean(axis=0), flat.std(axis=0)
    params = datagen.mlp_params(int(rng.integers(1 << 31)), scale=0.5).astype(np.float32)
    return f, pairs, params, mu.astype(np.float32), np.maximum(sd, 1e-3).astype(np.float32)


class _Owned(dict):
    """A state whose tables and networks are released with it."""

    def __del__(self):
        for h in [*self.get("tables", ()), self.get("mlp")]:
            if h is not None:
                h.free()


def prepare(case, seed):
    dev = torch.device("cuda")
    st = _Owned(case=case, seed=seed)
    kind = case["kind"]
    if kind == "mlp":
        f, pairs, params, mu, sd = _samples(case, seed)
        st.update(feats=torch.from_numpy(f).to(dev), pairs=torch.from_numpy(pairs).to(dev), params=params, mu=mu,
                  sd=sd, mlp=bnos.Mlp())
        st["mlp"].set_params(params, mu, sd)
        if case["op"] == "forward":
            st["logits"] = torch.empty(f.shape[:2], dtype=torch.float32, device=dev)
        elif case["op"] == "grad":
            st["grad"] = torch.empty(params.size, dtype=torch.float32, device=dev)
            st["loss"] = torch.empty(1, dtype=torch.float64, device=dev)
        else:
            steps = case["epochs"] * -(-case["rows"] // case["batch"])
            st["losses"] = torch.empty(steps, dtype=torch.float32, device=dev)
        return st
    if kind == "build":
        net, prior = _dataset(case, seed)
        st.update(data=net.data, arities=net.arities, prior=prior)
        if case["orders"]:
            _order_buffers(st, case["n"], case["orders"], True, seed, dev)
        return st
    if kind == "score":
        net, prior = _dataset(case, seed)
        st["tables"] = [bnos.build_score_table(net.data, net.arities, case["K"], prior=prior)]
        _order_buffers(st, case["n"], case["orders"], case["nodes"], seed, dev)
        if case["entry"] == "host":
            st["host_order"] = datagen.random_orders(case["n"], 1, seed + 2)[0]
        return st
    tables, states = [], []
    for d, (n, N) in enumerate(_dims(case)):
        net, prior = _dataset(case, seed + 31 * d, n, N)
        t = bnos.build_score_table(net.data, net.arities, min(case["K"], n - 1), prior=prior)
        tables.append(t)
        states.append(t.new_chain_state(case["chains"], case["iterations"], flags=True, topk=case["topk"]))
    st.update(tables=tables, states=states)
    if case["learned"]:
        feat = tables[0].node_features()
        mu = np.concatenate([[0.5, feat[:, 2].mean(), 10.0], feat.mean(axis=0)]).astype(np.float32)
        sd = np.concatenate([[0.3, feat[:, 2].std() + 1.0, 20.0], feat.std(axis=0) + 1e-3]).astype(np.float32)
        st["mlp"] = bnos.Mlp()
        st["mlp"].set_params(datagen.mlp_params(seed, scale=0.5).astype(np.float32), mu, sd)
    return st


def _order_buffers(st, n, B, nodes, seed, dev):
    st["orders"] = torch.from_numpy(datagen.random_orders(n, B, seed + 2)).to(dev)
    st["lse"] = torch.empty(B, dtype=torch.float64, device=dev)
    st["maxs"] = torch.empty(B, dtype=torch.float64, device=dev)
    st["best"] = torch.empty((B, n), dtype=torch.int64, device=dev)
    st["node_lse"] = torch.empty((B, n), dtype=torch.float64, device=dev) if nodes else None
    st["node_second"] = torch.empty((B, n), dtype=torch.float32, device=dev) if nodes else None


def _scored(st):
    out = dict(lse=st["lse"], maxs=st["maxs"], best=st["best"])
    if st["node_lse"] is not None:
        out.update(node_lse=st["node_lse"], node_second=st["node_second"])
    return out


# ------------------------------------------------------------------ one pass

def run(state):
    case = state["case"]
    kind = case["kind"]
    if kind == "mlp":
        m = state["mlp"]
        if case["op"] == "forward":
            m.forward(state["feats"], state["logits"])
            return dict(logits=state["logits"])
        if case["op"] == "grad":
            m.grad(state["feats"], state["pairs"], state["grad"], state["loss"])
            return dict(grad=state["grad"], loss=state["loss"])
        m.set_params(state["params"], state["mu"], state["sd"])
        m.train(state["feats"], state["pairs"], case["epochs"], case["batch"], 1e-3, seed=state["seed"],
                loss_trace=state["losses"])
        return dict(params=m.get_params()[0], losses=state["losses"])
    if kind == "build":
        t = bnos.build_score_table(state["data"], state["arities"], case["K"], prior=state["prior"])
        try:
            if case["orders"]:
                t.score_orders(state["orders"], state["lse"], state["maxs"], state["best"], state["node_lse"],
                               state["node_second"])
                return _scored(state)
            rows = [t.export(i) for i in range(case["n"])]
            return dict(masks=np.stack([m for m, _ in rows]), scores=np.stack([s for _, s in rows]),
                        features=t.node_features())
        finally:
            t.free()
    if kind == "score":
        t = state["tables"][0]
        if case["entry"] == "host":
            lse, mx, best = t.score_order(state["host_order"])
            return dict(lse=lse, maxs=mx, best=best)
        score = t.score_orders if case["entry"] == "device" else t.score_orders_noalloc
        score(state["orders"], state["lse"], state["maxs"], state["best"], state["node_lse"], state["node_second"])
        return _scored(state)
    states = state["states"]
    kw = dict(iterations=case["iterations"], seed=state["seed"], target=case["target"], mlp=state.get("mlp"))
    if case["tables"] == 1:
        state["tables"][0].run_chains(states[0], **kw)
    else:
        bnos.run_chains_multi(state["tables"], states, **kw)
    return [{k: v for k, v in s.items() if v is not None} for s in states]


# ------------------------------------------------------------------ what a pass cannot do without

def _sets(m, k):
    return sum(math.comb(m, j) for j in range(min(m, k) + 1))


def work(case):
    """Inputs read once, outputs written once; the counting or arithmetic that defines the result."""
    kind, n = case["kind"], case["n"]
    if kind == "mlp":
        nodes = case["rows"] * n
        fwd = 2 * nodes * (8 * 128 + 128 * 128 + 128)
        io = nodes * 32
        if case["op"] == "forward":
            return dict(bytes=io + nodes * 4, flops=fwd)
        passes = case.get("epochs", 1)
        return dict(bytes=passes * (io + case["rows"] * 8) + 2 * 17793 * 4, flops=passes * 3 * fwd)
    K = case["K"]
    if kind == "build":
        out = n * _sets(n - 1, K) * 12 if not case["orders"] else case["orders"] * (n * 20 + 16)
        return dict(bytes=case["N"] * n + out, flops=case["N"] * (_sets(n, K + 1) - 1))
    if kind == "score":
        B = case["orders"]
        return dict(bytes=B * (n * 4 + 16 + n * 8 + (n * 12 if case["nodes"] else 0)), flops=B * n)
    # each iteration reads and rewrites every chain's order and writes its score and flag
    chain_steps = case["chains"] * case["tables"] * case["iterations"]
    return dict(bytes=chain_steps * (8 * n + 9), flops=chain_steps * n)


# ------------------------------------------------------------------ the results in 64 bits

def _exact_rows(net, prior, K):
    """Local scores [n][S] in 64 bits (BDeu with sample size 1 plus the prior terms), a row's entries
    in ascending order of the parent mask with the node's own bit removed; and the masks [n][S] (node bits)."""
    n, N = net.n, net.N
    dev = torch.device("cuda")
    ar = torch.from_numpy(net.arities.astype(np.int64)).to(dev)
    data = torch.from_numpy(np.ascontiguousarray(net.data.T)).to(dev).long()
    combos = [torch.zeros((1, 0), dtype=torch.long)] + [
        torch.combinations(torch.arange(n - 1), r=j) for j in range(1, min(K, n - 1) + 1)]
    slots = torch.cat([torch.nn.functional.pad(c, (0, K - c.shape[1]), value=-1) for c in combos])
    key = torch.where(slots >= 0, 1 << slots.clamp(min=0), 0).sum(dim=1)
    slots = slots[torch.argsort(key)].to(dev)
    S = slots.shape[0]
    out = torch.empty((n, S), dtype=torch.float64, device=dev)
    masks = torch.empty((n, S), dtype=torch.long, device=dev)
    w = None if prior is None else torch.from_numpy(prior.astype(np.float64)).to(dev)
    for i in range(n):
        ids = torch.where(slots >= i, slots + 1, slots)
        live = slots >= 0
        masks[i] = torch.where(live, 1 << ids.clamp(min=0), 0).sum(dim=1)
        ids = ids.clamp(min=0)
        r = torch.where(live, ar[ids], 1)
        q = r.prod(dim=1)
        ri = int(ar[i])
        qcap = int(q.max())
        step = max(1, min(S, (1 << 26) // max(N, qcap * ri)))
        for f0 in range(0, S, step):
            f1 = min(S, f0 + step)
            k = torch.zeros((f1 - f0, N), dtype=torch.long, device=dev)
            for t in range(K):
                k = k * r[f0:f1, t:t + 1] + torch.where(live[f0:f1, t:t + 1], data[ids[f0:f1, t]], 0)
            flat = k * ri + data[i]
            one = torch.ones((), dtype=torch.float64, device=dev).expand(f1 - f0, N)
            nijk = torch.zeros((f1 - f0, qcap * ri), dtype=torch.float64, device=dev).scatter_add_(1, flat, one)
            nij = nijk.view(f1 - f0, qcap, ri).sum(dim=2)
            qf = q[f0:f1, None].double()
            a, b = 1.0 / (qf * ri), 1.0 / qf
            out[i, f0:f1] = ((torch.lgamma(nijk + a) - torch.lgamma(a)).sum(dim=1)
                             - (torch.lgamma(nij + b) - torch.lgamma(b)).sum(dim=1))
        if w is not None:
            term = math.log(10.0) * 100.0 * (w[i] * 0.5) ** 3
            out[i] += torch.where(live, term[ids], 0.0).sum(dim=1)
    return out, masks


def _exact_orders(rows, masks, orders):
    n = rows.shape[0]
    dev = rows.device
    B = orders.shape[0]
    nl = torch.empty((B, n), dtype=torch.float64, device=dev)
    nm, ns = nl.clone(), nl.clone()
    for b in range(B):
        seen = 0
        for v in orders[b]:
            x = torch.where((masks[v] & ~seen) == 0, rows[v], -math.inf)
            nl[b, v] = torch.logsumexp(x, 0)
            top = torch.topk(x, min(2, x.numel())).values
            nm[b, v] = top[0]
            ns[b, v] = top[1] if top.numel() > 1 else -math.inf
            seen |= 1 << int(v)
    return nl.cpu().numpy(), nm.cpu().numpy(), ns.cpu().numpy()


def _exact_mlp_loss(p, z, pairs, eps):
    """(logits, mean -ln q of the pairs) of flat 64-bit parameters on normalised features z."""
    H, F = 128, 8
    cut = np.cumsum([H * F, H, H * H, H, H])
    W1, b1, W2, b2, w3, b3 = [p[a:b] for a, b in zip([0, *cut], [*cut, p.numel()])]
    h = torch.relu(torch.relu(z @ W1.view(H, F).T + b1) @ W2.view(H, H).T + b2)
    logit = h @ w3 + b3
    if pairs is None:
        return logit, None
    n = z.shape[1]
    s = torch.softmax(logit, dim=1)
    pa, pb = s.gather(1, pairs[:, :1])[:, 0], s.gather(1, pairs[:, 1:])[:, 0]
    q = (1 - eps) * pa * pb * (1 / (1 - pa) + 1 / (1 - pb)) + eps * 2 / (n * (n - 1))
    return logit, -torch.log(q).mean()


def _mix(z):
    m = (1 << 64) - 1
    z = ((z ^ (z >> 30)) * 0xBF58476D1CE4E5B9) & m
    z = ((z ^ (z >> 27)) * 0x94D049BB133111EB) & m
    return z ^ (z >> 31)


def _exact_mlp(case, seed):
    f, pairs, params, mu, sd = _samples(case, seed)
    dev = torch.device("cuda")
    z = (torch.from_numpy(f).to(dev).double() - torch.from_numpy(mu).to(dev).double()) / torch.from_numpy(sd).to(dev).double()
    pr = torch.from_numpy(pairs).to(dev).long()
    p = torch.from_numpy(params).to(dev).double()
    eps = float(np.float32(0.1))
    if case["op"] == "forward":
        return dict(logits=_exact_mlp_loss(p, z, None, eps)[0].cpu().numpy())
    p.requires_grad_(True)
    if case["op"] == "grad":
        loss = _exact_mlp_loss(p, z, pr, eps)[1]
        loss.backward()
        return dict(grad=p.grad.cpu().numpy(), loss=loss.detach().reshape(1).cpu().numpy())
    # Adam over the epochs' visiting orders: sample (offset + j * stride) mod count at place j
    count, batch = case["rows"], min(case["batch"], case["rows"])
    m, v = torch.zeros_like(p), torch.zeros_like(p)
    losses, t = [], 0
    for ep in range(case["epochs"]):
        r = _mix(seed ^ _mix(0x5EED + ep))
        stride = 1 + r % count
        while math.gcd(stride, count) != 1:
            stride = stride % count + 1
        offset = _mix(r) % count
        for b in range(0, count, batch):
            j = (torch.arange(b, min(b + batch, count), device=dev) * stride + offset) % count
            loss = _exact_mlp_loss(p, z[j], pr[j], eps)[1]
            g, = torch.autograd.grad(loss, p)
            losses.append(float(loss))
            t += 1
            m = 0.9 * m + 0.1 * g
            v = 0.999 * v + 0.001 * g * g
            with torch.no_grad():
                p -= 1e-3 * (m / (1 - 0.9 ** t)) / (torch.sqrt(v / (1 - 0.999 ** t)) + 1e-8)
    return dict(params=p.detach().cpu().numpy(), losses=np.array(losses))


def exact(case, seed):
    kind = case["kind"]
    if kind == "mlp":
        return _exact_mlp(case, seed)
    if kind == "chains":                   # a trajectory of accept decisions has no 64-bit value of its own
        return None
    n, K = case["n"], case["K"]
    if n * _sets(n - 1, K) * case["N"] > 1.0e10:   # the 60-node tables take minutes this way
        return None
    net, prior = _dataset(case, seed)
    rows, masks = _exact_rows(net, prior, K)
    if kind == "build" and not case["orders"]:
        host = rows.cpu().numpy()
        term = np.zeros((n, n)) if prior is None else math.log(10.0) * 100.0 * (prior.astype(np.float64) * 0.5) ** 3
        np.fill_diagonal(term, 0.0)
        feat = np.stack([term.sum(axis=1), term.sum(axis=0), host.max(axis=1), host.mean(axis=1), host.std(axis=1)], axis=1)
        return dict(masks=None, scores=host, features=feat)
    orders = datagen.random_orders(n, case["orders"], seed + 2)
    nl, nm, ns = _exact_orders(rows, masks, orders)
    if kind == "score" and case["entry"] == "host":
        return dict(lse=float(nl.sum()), maxs=float(nm.sum()), best=None)
    out = dict(lse=nl.sum(axis=1), maxs=nm.sum(axis=1), best=None)
    if kind == "build" or case["nodes"]:
        out.update(node_lse=nl, node_second=ns)
    return out
