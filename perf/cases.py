"""Performance cases of the library: the calls a track-finding program makes,
through the public entry points of ``paper_2402_09633_amd.gnn``.

Each case is one step of the pipeline on one event (or a few queued events):
edge scoring by the interaction network at the three arithmetic settings a
user can choose, the request queue, the edge filter, the embedding, the
fixed-radius search and the track candidates (connected components).  Inputs
are synthetic hit graphs with the geometry of ``inputs.layered_graph``, built
on the device so that they are quick to make, and cut to an exact edge count.
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_2402_09633_amd import gnn as G
from paper_2402_09633_amd import inputs as I

DEV = "cuda"
F = 3  # raw features of a hit: r, phi, z


# ------------------------------------------------------------------ cases ---

def _infer(name, hits, edges, hidden, iters, dtype, sets=1, order="source"):
    return {"name": name, "op": "infer", "hits": hits, "edges": edges, "hidden": hidden,
            "iters": iters, "dtype": dtype, "sets": sets, "order": order}


def listed():
    return [
        # The event size of the paper's introduction (about 300k hits and 1M
        # edges), the step that this library exists for: fp32, the default.
        _infer("full_fp32", 300_000, 1_000_513, 128, 8, "fp32"),
        # The same event with the bf16 model (hi/lo bf16 weights).
        _infer("full_bf16", 300_000, 1_000_513, 128, 8, "bf16"),
        # The same with fp16 weights, the setting a service tuned for
        # throughput runs.
        _infer("full_f16w", 300_000, 1_000_513, 128, 8, "f16w"),
        # A mid-size event (low pile-up, or one detector region).
        _infer("mid_fp32", 50_000, 329_756, 128, 8, "fp32"),
        # A small ragged event: narrow model, one weight pair per iteration,
        # edges in no particular order (as a graph builder may emit them).
        _infer("ragged_bf16", 20_011, 70_001, 64, 4, "bf16", sets=4, order="shuffled"),
        # The smallest calls: a region of interest of 2,000 hits, where
        # latency is what a user sees.
        _infer("tiny_fp32", 2_000, 8_000, 64, 2, "fp32"),
        # A service: ragged events queued at once in front of several model
        # instances on one GPU.
        {"name": "serve_f16w", "op": "serve", "hits": 30_000, "edges": 100_003, "hidden": 128,
         "iters": 8, "dtype": "f16w", "events": 4, "instances": 4},
        # The step before the network: filter MLP over the candidate edges of
        # a full event, and the kept edges as a new edge list.
        {"name": "filter_full", "op": "filter", "hits": 300_000, "edges": 2_000_003, "hidden": 64},
        # Graph construction: embedding of a full event's hits ...
        {"name": "embed_full", "op": "embed", "hits": 300_000, "hidden": 128, "dim": 8},
        # ... and the pairs within the radius in the embedded space.
        {"name": "frnn_full", "op": "frnn", "hits": 300_000, "dim": 8, "radius": 0.02},
        # The step after the network: track candidates of a full event from
        # the scores a trained model gives (most true segments kept, few
        # false ones).
        {"name": "wcc_tracks", "op": "wcc", "hits": 300_000, "edges": 1_000_513, "keep": 0.9,
         "fake": 0.02},
        # The same step at a loose working point (every edge kept): the event
        # collapses into large components.
        {"name": "wcc_loose", "op": "wcc", "hits": 150_001, "edges": 500_009, "keep": 1.0,
         "fake": 1.0},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    op = rng.choice(["infer"] * 6 + ["serve", "filter", "embed", "frnn", "wcc"])
    hits = _log_int(rng, 500, 300_000)
    hidden = rng.choice([64, 128, 128])
    if op == "infer":
        iters = rng.randint(1, 8)
        edges = min(int(hits * rng.uniform(1.0, 6.0)), 1_000_000)
        return {"op": op, "hits": hits, "edges": edges, "hidden": hidden, "iters": iters,
                "dtype": rng.choice(["fp32", "bf16", "f16w"]), "sets": rng.choice([1, 1, iters]),
                "order": rng.choice(["source", "source", "shuffled"])}
    if op == "serve":
        hits = _log_int(rng, 500, 60_000)
        return {"op": op, "hits": hits, "edges": int(hits * rng.uniform(1.0, 4.0)),
                "hidden": hidden, "iters": rng.randint(1, 8),
                "dtype": rng.choice(["fp32", "bf16", "f16w"]), "events": rng.randint(2, 4),
                "instances": rng.randint(1, 4)}
    if op == "filter":
        return {"op": op, "hits": hits, "edges": int(hits * rng.uniform(1.0, 6.6)),
                "hidden": hidden}
    if op == "embed":
        return {"op": op, "hits": hits, "hidden": hidden, "dim": rng.randint(3, 16)}
    if op == "frnn":
        return {"op": op, "hits": hits, "dim": rng.randint(3, 12),
                "radius": rng.choice([0.01, 0.015, 0.02])}
    return {"op": op, "hits": hits, "edges": int(hits * rng.uniform(1.0, 4.0)),
            "keep": round(rng.uniform(0.5, 1.0), 2), "fake": round(rng.uniform(0.0, 0.1), 3)}


# ----------------------------------------------------------------- inputs ---

def _hits(n, rng):
    """Hits on 10 cylinders, layer-major: features [n][3] and (phi, z, layer offsets)."""
    per = [n // I.N_LAYERS] * I.N_LAYERS
    for k in range(n - sum(per)):
        per[I.N_LAYERS - 1 - k] += 1
    r = np.repeat(I.R_MIN_MM * (I.R_MAX_MM / I.R_MIN_MM) **
                  (np.arange(I.N_LAYERS) / (I.N_LAYERS - 1)), per)
    phi = rng.uniform(-math.pi, math.pi, n)
    z = rng.normal(0.0, I.Z_SIGMA_MM, n)
    x = np.stack([r / 1000.0, phi / math.pi, z / 1000.0], axis=1).astype(np.float32)
    offs = np.concatenate([[0], np.cumsum(per)]).tolist()
    return (torch.as_tensor(x).to(DEV), torch.as_tensor(phi).to(DEV), torch.as_tensor(z).to(DEV),
            offs)


def _segments(phi, z, offs, dphi, dz):
    """Edges to the next layer inside the windows, at most 8 per hit (the
    smallest |dphi|), grouped by source."""
    srcs, dsts = [], []
    for l in range(I.N_LAYERS - 1):
        a, b = slice(offs[l], offs[l + 1]), slice(offs[l + 1], offs[l + 2])
        pa = phi[a]
        ps, order = torch.sort(phi[b])
        nb = ps.numel()
        if pa.numel() == 0 or nb == 0:
            continue
        ext = torch.cat([ps - 2 * math.pi, ps, ps + 2 * math.pi])
        lo = torch.searchsorted(ext, pa - dphi, right=True)
        hi = torch.minimum(torch.searchsorted(ext, pa + dphi), lo + nb)
        cnt = hi - lo
        ia = torch.repeat_interleave(torch.arange(pa.numel(), device=DEV), cnt)
        first = torch.cumsum(cnt, 0) - cnt
        pos = torch.arange(ia.numel(), device=DEV) - first[ia] + lo[ia]
        gi, gj = ia + offs[l], order[pos % nb] + offs[l + 1]
        ad = (ext[pos] - phi[gi]).abs()
        ok = (z[gj] - z[gi]).abs() < dz
        gi, gj, ad = gi[ok], gj[ok], ad[ok]
        o = torch.argsort(ad, stable=True)
        o = o[torch.argsort(gi[o], stable=True)]
        gi, gj = gi[o], gj[o]
        k = torch.arange(gi.numel(), device=DEV)
        start = torch.searchsorted(gi, gi)
        sel = k - start < I.MAX_OUT_DEGREE
        srcs.append(gi[sel])
        dsts.append(gj[sel])
    return torch.cat(srcs), torch.cat(dsts)


def _event(hits, edges, seed, order="source"):
    """(x [hits][3], edge_index [2][edges]) of one event: windows as wide as
    the edge count needs, then a seeded choice of exactly that many edges."""
    rng = np.random.default_rng(seed)
    x, phi, z, offs = _hits(hits, rng)
    # windows whose mean out-degree is the one asked for, a little widened
    want = 1.08 * edges / (0.9 * hits)
    s = 1.0
    for _ in range(40):
        got = hits / 10 * s * I.DPHI_MID / math.pi * math.erf(s * I.DZ_MID / (2 * I.Z_SIGMA_MM))
        s = min(s * math.sqrt(want / max(got, 1e-9)), 2.0 / I.DPHI_MID)
    while True:
        src, dst = _segments(phi, z, offs, s * I.DPHI_MID, s * I.DZ_MID)
        if src.numel() >= edges:
            break
        s *= 1.15
    pick = rng.permutation(src.numel())[:edges]
    if order == "source":
        pick.sort()
    pick = torch.as_tensor(pick).to(DEV)
    return x, torch.stack([src[pick], dst[pick]]).to(torch.int32).contiguous()


def _weights(case, seed):
    return I.make_weights(F, case["hidden"], case.get("sets", 1), seed, affine_noise=0.1)


def _model(case, seed):
    dtype = G.GNN_FP32 if case["dtype"] == "fp32" else G.GNN_BF16
    flags = G.GNN_F16_WEIGHTS if case["dtype"] == "f16w" else 0
    return G.Model(_weights(case, seed), G.make_dims(F, case["hidden"], case["iters"],
                                                     case.get("sets", 1), dtype, flags=flags))


def _serve_sizes(case):
    """Ragged sizes around the case's, one event each."""
    n = case["events"]
    f = [0.7 + 0.6 * k / max(1, n - 1) for k in range(n)]
    return [(int(case["hits"] * v), int(case["edges"] * v)) for v in f]


def _threshold(scores):
    """A working point near the median that no score is close to: the middle
    of the widest gap between neighbouring scores of the central tenth."""
    s = torch.sort(scores).values
    mid = s[int(0.45 * s.numel()):int(0.55 * s.numel()) + 2]
    k = int(torch.argmax(mid[1:] - mid[:-1]))
    return float((mid[k] + mid[k + 1]) / 2)


def _track_scores(ei, case, rng):
    """Scores of a trained model: one true continuation per hit scores high,
    the rest low, apart from the lost and the false ones."""
    src = ei[0].cpu().numpy()
    n = src.size
    true = np.zeros(n, bool)
    o = rng.permutation(n)
    _, first = np.unique(src[o], return_index=True)
    true[o[first]] = True
    high = np.where(true, rng.random(n) < case["keep"], rng.random(n) < case["fake"])
    s = np.where(high, 1.0 - 0.45 * rng.random(n) ** 2, 0.45 * rng.random(n) ** 2)
    return torch.as_tensor(s.astype(np.float32)).to(DEV)


class _Filter:
    """One filter handle, destroyed with the object."""

    def __init__(self, case, seed):
        self.handle = G.gnn_filter_create(I.make_filter_weights(F, case["hidden"], seed, 0.1),
                                          G.make_filter_dims(F, case["hidden"]))

    def __del__(self):
        G.gnn_filter_destroy(self.handle)


class _Service:
    """A model and its request queue, closed in that order."""

    def __init__(self, case, seed):
        self.model = _model(case, seed)
        self.server = G.Server(self.model, case["instances"])

    def __del__(self):
        self.server.close()
        self.model.close()


def _points(case, seed):
    return I.clustered_points(case["hits"], case["dim"], seed, sigma=case["radius"] / 4)


def prepare(case, seed):
    op = case["op"]
    s = {"op": op}
    if op == "infer":
        s["x"], s["ei"] = _event(case["hits"], case["edges"], seed, case["order"])
        s["model"] = _model(case, seed + 7)
        s["out"] = torch.empty(case["edges"], dtype=torch.float32, device=DEV)
    elif op == "serve":
        s["events"] = [_event(h, e, seed + 1000 * k)
                       for k, (h, e) in enumerate(_serve_sizes(case))]
        s["service"] = _Service(case, seed + 7)
        s["out"] = [torch.empty(ei.shape[1], dtype=torch.float32, device=DEV)
                    for _, ei in s["events"]]
    elif op == "filter":
        s["x"], s["ei"] = _event(case["hits"], case["edges"], seed)
        s["filter"] = _Filter(case, seed + 7)
        s["threshold"] = _threshold(_exact_filter(case, seed, s["x"], s["ei"]))
        s["scores"] = torch.empty(case["edges"], dtype=torch.float32, device=DEV)
        s["kept"] = torch.zeros(2 * case["edges"], dtype=torch.int32, device=DEV)
    elif op == "embed":
        s["x"] = _hits(case["hits"], np.random.default_rng(seed))[0]
        s["model"] = G.Embedder(I.make_embed_weights(F, case["hidden"], case["dim"], seed + 7, 0.1),
                                G.make_embed_dims(F, case["hidden"], case["dim"]))
        s["z"] = torch.empty(case["hits"], case["dim"], dtype=torch.float32, device=DEV)
    elif op == "frnn":
        s["z"] = torch.as_tensor(_points(case, seed)).to(DEV)
        s["r2"] = case["radius"] ** 2
        s["room"] = 16 * case["hits"]
        s["pairs"] = torch.zeros(2 * s["room"], dtype=torch.int32, device=DEV)
    elif op == "wcc":
        x, s["ei"] = _event(case["hits"], case["edges"], seed)
        s["n"] = case["hits"]
        s["scores"] = _track_scores(s["ei"], case, np.random.default_rng(seed + 3))
        s["labels"] = torch.empty(case["hits"], dtype=torch.int32, device=DEV)
    return s


# -------------------------------------------------------------------- run ---

def run(state):
    op = state["op"]
    if op == "infer":
        return state["model"](state["x"], state["ei"], out=state["out"], logits=True)
    if op == "serve":
        server = state["service"].server
        ids = [server.submit(x, ei, out) for (x, ei), out in zip(state["events"], state["out"])]
        for i in ids:
            server.wait(i)
        return state["out"]
    if op == "filter":
        x, ei = state["x"], state["ei"]
        n = G.gnn_filter_apply(state["filter"].handle, x, ei, x.shape[0], ei.shape[1],
                               state["threshold"], state["scores"], state["kept"])
        return [state["scores"], state["kept"], n]
    if op == "embed":
        return state["model"](state["x"], state["z"])
    if op == "frnn":
        z = state["z"]
        n = G.gnn_frnn(z, z.shape[0], z.shape[1], state["r2"], state["pairs"], state["room"])
        return [state["pairs"], n]
    G.gnn_wcc(state["ei"], state["scores"], 0.5, state["n"], state["ei"].shape[1],
              state["labels"])
    return state["labels"]


# ------------------------------------------------------------------- work ---

def _infer_work(case, hits, edges):
    """The network with its edge-side first layers regrouped per node, the
    cheapest exact form: inputs, weights and scores once, 2 operations per
    multiply-add."""
    H, T = case["hidden"], case["iters"]
    per_node = F * H + H * H + 2 * H * H * (T + 2) + T * 4 * H * H
    per_edge = H * H + T * 2 * H * H + H * H + H
    return {"bytes": 4 * (hits * F + 3 * edges + I.weight_count(F, H, case.get("sets", 1))),
            "flops": 2.0 * (hits * per_node + edges * per_edge)}


def work(case):
    op, n, H = case["op"], case["hits"], case.get("hidden", 0)
    if op == "infer":
        return _infer_work(case, n, case["edges"])
    if op == "serve":
        w = [_infer_work(case, h, e) for h, e in _serve_sizes(case)]
        return {k: sum(v[k] for v in w) for k in ("bytes", "flops")}
    if op == "filter":
        e = case["edges"]
        # indices in, scores out, half of the edges kept
        return {"bytes": 4 * (n * F + 2 * e + e + e), "flops": 2.0 * e * (2 * F * H + H * H + H)}
    if op == "embed":
        return {"bytes": 4 * n * (F + case["dim"]),
                "flops": 2.0 * n * (F * H + H * H + H * case["dim"])}
    if op == "frnn":
        # points in, about two pairs per point out; a distance per pair
        return {"bytes": 4 * n * case["dim"] + 16 * n, "flops": 6.0 * n * case["dim"]}
    return {"bytes": 12 * case["edges"] + 4 * n, "flops": 0.0}


def tolerance(case):
    op = case["op"]
    if op in ("frnn", "wcc"):
        return "exact"
    # Four times the error measured against 64 bits (full event: logits 1.1e-6
    # in fp32, 1.1e-2 in the 16-bit models, whose rounding of one row travels
    # through every later layer; served scores 2.9e-3; embedding 2.2e-7).
    if op == "infer":
        return {"rel": 5e-6, "max": 1e-3} if case["dtype"] == "fp32" else {"rel": 3e-2, "max": 0.6}
    if op == "serve":
        return {"rel": 5e-6, "max": 1e-3} if case["dtype"] == "fp32" else {"rel": 1.2e-2, "max": 0.2}
    return {"rel": 1e-6, "max": 1e-4}


# ------------------------------------------------------------------ exact ---

def _views(blob, views):
    return {k: torch.as_tensor(v.astype(np.float64)).to(DEV) for k, v in views.items()}


def _phi(p, name, a):
    y = a @ p[name + ".W"].T + p[name + ".b"]
    y = torch.nn.functional.layer_norm(y, (y.shape[1],), p[name + ".g"], p[name + ".beta"], 1e-5)
    return torch.relu(y)


def _mlp(p, name, a):
    return _phi(p, name + ".1", _phi(p, name + ".0", a))


def _rows(f, n, step=1 << 17):
    return torch.cat([f(slice(i, min(n, i + step))) for i in range(0, n, step)])


def _exact_logits(case, seed, x, ei):
    blob = _weights(case, seed)
    p = _views(blob, I.blob_views(blob, F, case["hidden"], case.get("sets", 1)))
    s, d = ei[0].long(), ei[1].long()
    n, m = x.shape[0], s.numel()
    h = _mlp(p, "node_enc", x.double())
    e = _rows(lambda r: _mlp(p, "edge_enc", torch.cat([h[s[r]], h[d[r]]], 1)), m)
    for t in range(case["iters"]):
        k = 0 if case.get("sets", 1) == 1 else t
        e = _rows(lambda r: _mlp(p, "edge_mlp%d" % k, torch.cat([h[s[r]], h[d[r]], e[r]], 1)), m)
        agg_in = torch.zeros_like(h).index_add_(0, d, e)
        agg_out = torch.zeros_like(h).index_add_(0, s, e)
        h = _rows(lambda r: _mlp(p, "node_mlp%d" % k, torch.cat([h[r], agg_in[r], agg_out[r]], 1)),
                  n)
    return _rows(lambda r: (_phi(p, "edge_cls.0", torch.cat([h[s[r]], h[d[r]], e[r]], 1))
                            @ p["edge_cls.1.W"].T + p["edge_cls.1.b"])[:, 0], m)


def _exact_filter(case, seed, x, ei):
    blob = I.make_filter_weights(F, case["hidden"], seed + 7, 0.1)
    p = _views(blob, I.filter_blob_views(blob, F, case["hidden"]))
    xd, s, d = x.double(), ei[0].long(), ei[1].long()
    return _rows(lambda r: torch.sigmoid(
        _mlp(p, "filter", torch.cat([xd[s[r]], xd[d[r]]], 1)) @ p["filter.2.W"].T
        + p["filter.2.b"])[:, 0], s.numel(), 1 << 19)


def exact(case, seed):
    op = case["op"]
    if op == "infer":
        x, ei = _event(case["hits"], case["edges"], seed, case["order"])
        return _exact_logits(case, seed + 7, x, ei)
    if op == "serve":
        return [torch.sigmoid(_exact_logits(case, seed + 7, *_event(h, e, seed + 1000 * k)))
                for k, (h, e) in enumerate(_serve_sizes(case))]
    if op == "filter":
        x, ei = _event(case["hits"], case["edges"], seed)
        return [_exact_filter(case, seed, x, ei), None, None]
    if op == "embed":
        x = _hits(case["hits"], np.random.default_rng(seed))[0].double()
        blob = I.make_embed_weights(F, case["hidden"], case["dim"], seed + 7, 0.1)
        p = _views(blob, I.embed_blob_views(blob, F, case["hidden"], case["dim"]))
        return _mlp(p, "embed", x) @ p["embed.2.W"].T + p["embed.2.b"]
    return None  # pairs and labels are whole numbers
