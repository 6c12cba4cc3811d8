"""The work that a user of this framework has it do, as cases that can be timed.

Every case is a dict of plain values; `prepare` makes what a program holds
before the call (inputs, output buffers, workspaces), `run` makes one pass
through the public entry points of paper_1003_3684_amd.native.  The kinds:

  kron_csr       a Kronecker graph and its CSR in one call: the benchmark's step
  pba_csr        a PBA graph, then its symmetrized CSR
  csr            an edge list that the program already has, made into a CSR
  stats          degree histogram, tail exponent and wedge closure of a graph
  ensemble       many PBA and Kronecker graphs of the ensemble recipe, summarised
  paths          path lengths from a sample of sources over a symmetric CSR
  mlp_train      one step of the surrogate's training loop
  mlp_eval       the surrogate's value and its gradient in the input features
  randomized_pk  the two randomizations of the Kronecker power, and the block
                 matrix of the first
"""
import ctypes
import math

import numpy as np
import torch

from paper_1003_3684_amd import native as sfg
from paper_1003_3684_amd import workloads as wl

INITIATORS = {
    "2x2": (2, wl.KRON_K20["initiator"]),
    "3x3": (3, wl.KRON_SCALE_B["initiator"]),
    "3x3pad4": (4, wl.KRON_SCALE["initiator"]),
}
D_IN, D_OUT = 10, 34  # the surrogate's features and targets
ADAM_STEP = 100       # steps the training loop has made when the timed one comes


def listed():
    return [
        # The smallest graph of the ensemble recipe, made on its own: latency and launches.
        {"name": "kron_csr_k10", "kind": "kron_csr", "init": "2x2", "k": 10, "edges": 16 << 10, "id_bytes": 4, "flags": 0},
        # The 2x2 configuration at 20 levels, an ordinary graph.
        {"name": "kron_csr_k20", "kind": "kron_csr", "init": "2x2", "k": 20, "edges": 1 << 24, "id_bytes": 4, "flags": 0},
        # The benchmark's step (padded 3x3 initiator, 2^30 ids of 8 bytes) at a fifth of its edges.
        {"name": "kron_csr_k15_pad", "kind": "kron_csr", "init": "3x3pad4", "k": 15, "edges": 1 << 30, "id_bytes": 8, "flags": 0},
        # The small PBA configuration and its undirected CSR.
        {"name": "pba_csr_n65536", "kind": "pba_csr", "n": 65536, "m": 4, "parts": 64, "p": 0.1, "id_bytes": 4},
        # The large PBA configuration and its undirected CSR.
        {"name": "pba_csr_n2e27", "kind": "pba_csr", "n": 1 << 27, "m": 5, "parts": 1024, "p": 0.1, "id_bytes": 4},
        # An edge list from elsewhere (ragged sizes, 8-byte ids) made simple and undirected.
        {"name": "csr_simple_n3e6", "kind": "csr", "n": 3000017, "edges": 24000131, "id_bytes": 8, "flags": 3},
        # The statistics of one generated graph, as the exponent search asks for them.
        {"name": "stats_k14", "kind": "stats", "n": 1 << 14, "edges": 16 << 14, "id_bytes": 4, "samples": 2000},
        # A table of the ensemble recipe.
        {"name": "ensemble_96", "kind": "ensemble", "graphs": 96, "samples": 10000},
        # The sampled path statistics of a graph of two million vertices.
        {"name": "paths_n2e6", "kind": "paths", "n": 2000003, "edges": 16000000, "id_bytes": 4, "sources": 64},
        # The training step of the surrogate at its own batch and width.
        {"name": "mlp_train_b4096", "kind": "mlp_train", "batch": 4096, "width": 256, "hidden": 3},
        # The surrogate's inversion: a step for all of its restarts at once.
        {"name": "mlp_eval_b16", "kind": "mlp_eval", "batch": 16, "width": 256, "hidden": 3},
        # The randomized powers of a seed with the size of the paper's (5 vertices, 11 edges).
        {"name": "randomized_pk_k8", "kind": "randomized_pk", "k": 8, "edges0": 11, "p": 0.05, "random": 100000000,
         "blocks": 25, "id_bytes": 4},
    ]


def _log(rng, lo, hi):
    """A whole number between lo and hi, uniform in its logarithm."""
    return min(hi, int(lo * (hi / lo) ** rng.random()))


def draw(rng):
    kind = rng.choice(["kron_csr", "kron_csr", "pba_csr", "pba_csr", "csr", "csr", "stats", "ensemble", "paths",
                       "mlp_train", "mlp_eval", "randomized_pk"])
    if kind == "kron_csr":
        init = rng.choice(["2x2", "3x3", "3x3pad4"])
        n0 = INITIATORS[init][0]
        edges = _log(rng, 5000, 1 << 27)
        per_vertex = rng.uniform(1, 16) if init != "3x3pad4" else rng.uniform(0.5, 4)
        k = max(2, round(math.log(max(edges / per_vertex, 16), n0)))
        return {"kind": kind, "init": init, "k": k, "edges": edges, "id_bytes": rng.choice([4, 8]),
                "flags": rng.choice([0, 0, 1, 3])}
    if kind == "pba_csr":
        m = rng.randint(2, 8)
        n = _log(rng, 1000, (1 << 26) // m)
        parts = rng.choice([p for p in (1, 8, 64, 256, 1024) if 8 * p <= n])
        return {"kind": kind, "n": n, "m": m, "parts": parts, "p": round(rng.uniform(0.0, 0.5), 3), "id_bytes": rng.choice([4, 4, 8])}
    if kind == "csr":
        edges = _log(rng, 3000, 1 << 26)
        return {"kind": kind, "n": max(2, int(edges / rng.uniform(1, 16))), "edges": edges, "id_bytes": rng.choice([4, 8]),
                "flags": rng.choice([0, 1, 3])}
    if kind == "stats":
        edges = _log(rng, 10000, 1 << 24)
        return {"kind": kind, "n": max(64, edges // rng.randint(2, 16)), "edges": edges, "id_bytes": rng.choice([4, 4, 8]),
                "samples": rng.choice([2000, 10000])}
    if kind == "ensemble":
        return {"kind": kind, "graphs": _log(rng, 6, 160), "samples": rng.choice([2000, 10000])}
    if kind == "paths":
        edges = _log(rng, 20000, 1 << 24)
        return {"kind": kind, "n": max(64, edges // rng.randint(2, 16)), "edges": edges, "id_bytes": rng.choice([4, 4, 8]),
                "sources": rng.choice([1, 16, 64, 64, 100])}
    if kind == "mlp_train":
        return {"kind": kind, "batch": _log(rng, 100, 8192), "width": rng.choice([64, 128, 200, 256]), "hidden": rng.randint(2, 4)}
    if kind == "mlp_eval":
        return {"kind": kind, "batch": _log(rng, 1, 4096), "width": rng.choice([64, 128, 200, 256]), "hidden": rng.randint(2, 4)}
    return {"kind": kind, "k": rng.randint(4, 7), "edges0": rng.randint(8, 12), "p": round(rng.uniform(0.01, 0.1), 3),
            "random": _log(rng, 1000, 30000000), "blocks": rng.choice([5, 25, 125]), "id_bytes": rng.choice([4, 4, 8])}


# ----------------------------------------------------------------------------- inputs
def _gen(seed):
    return torch.Generator(device="cuda").manual_seed(int(seed))


def _dtype(id_bytes):
    return torch.int32 if id_bytes == 4 else torch.int64


def _rmat(n, edges, seed):
    """A skewed edge list over n vertices (int64): the R-MAT draw with the 2x2 configuration's cells, ids folded into
    [0, n)."""
    g = _gen(seed)
    levels = max(1, (n - 1).bit_length())
    u = torch.zeros(edges, dtype=torch.int64, device="cuda")
    v = torch.zeros_like(u)
    for _ in range(levels):
        x = torch.rand(edges, device="cuda", generator=g)
        row = x >= 0.76
        u = 2 * u + row
        v = 2 * v + (((x >= 0.57) & ~row) | (x >= 0.95))
    return u % n, v % n


def _vertices(case):
    return INITIATORS[case["init"]][0] ** case["k"]


def _seed_matrix(case, seed):
    """A 5x5 seed graph with edges0 edges, among them the loop at vertex 0."""
    r = np.random.default_rng(int(seed))
    W = np.zeros(25, np.float32)
    W[0] = 1
    W[1 + r.permutation(24)[:case["edges0"] - 1]] = 1
    return W.reshape(5, 5)


def _simple_csr(n, u, v, dtype):
    keep = u != v
    u, v = u[keep], v[keep]
    key = torch.unique(torch.cat([u * n + v, v * n + u]))
    row_ptr = torch.zeros(n + 1, dtype=torch.int64, device="cuda")
    row_ptr[1:] = torch.cumsum(torch.bincount(key // n, minlength=n), 0)
    return row_ptr, (key % n).to(dtype)


def _layers(case):
    dims = [D_IN] + [case["width"]] * case["hidden"] + [D_OUT]
    return list(zip(dims[:-1], dims[1:]))


def _params(case, g):
    parts = []
    for i, o in _layers(case):
        parts.append(torch.randn(i * o, device="cuda", generator=g) * math.sqrt(2.0 / i))
        parts.append(torch.randn(o, device="cuda", generator=g) * 0.05)
    return torch.cat(parts)


def _features(rows, g):
    """Rows as the surrogate's encoding has them: shares and scaled logarithms of order one."""
    return torch.rand(rows, D_IN, device="cuda", generator=g) * 1.5


# ----------------------------------------------------------------------------- prepare
def prepare(case, seed):
    kind = case["kind"]
    s = {"kind": kind, "case": case, "seed": int(seed)}
    if kind == "kron_csr":
        n, E, dt, flags = _vertices(case), case["edges"], _dtype(case["id_bytes"]), case["flags"]
        s["out"] = {"src": torch.empty(E, dtype=dt, device="cuda"), "dst": torch.empty(E, dtype=dt, device="cuda"),
                    "row_ptr": torch.empty(n + 1, dtype=torch.int64, device="cuda"),
                    "col": torch.zeros(2 * E if flags & 1 else E, dtype=dt, device="cuda"),
                    "ws": sfg.workspace(sfg.edges_to_csr_workspace_bytes(n, E, case["id_bytes"], flags))}
    elif kind == "pba_csr":
        n, E, dt = case["n"], case["n"] * case["m"], _dtype(case["id_bytes"])
        s["src"], s["dst"] = torch.empty(E, dtype=dt, device="cuda"), torch.empty(E, dtype=dt, device="cuda")
        s["row_ptr"] = torch.empty(n + 1, dtype=torch.int64, device="cuda")
        s["col"] = torch.empty(2 * E, dtype=dt, device="cuda")
        s["ws"] = sfg.workspace(max(sfg.pba_workspace_bytes(n, case["m"], case["parts"]),
                                    sfg.edges_to_csr_workspace_bytes(n, E, case["id_bytes"], 1)))
    elif kind == "csr":
        n, E, dt, flags = case["n"], case["edges"], _dtype(case["id_bytes"]), case["flags"]
        u, v = _rmat(n, E, seed)
        s["src"], s["dst"] = u.to(dt), v.to(dt)
        s["row_ptr"] = torch.empty(n + 1, dtype=torch.int64, device="cuda")
        s["col"] = torch.zeros(2 * E if flags & 1 else E, dtype=dt, device="cuda")
        s["ws"] = sfg.workspace(sfg.edges_to_csr_workspace_bytes(n, E, case["id_bytes"], flags))
    elif kind == "stats":
        u, v = _rmat(case["n"], case["edges"], seed)
        s["src"], s["dst"] = u.to(_dtype(case["id_bytes"])), v.to(_dtype(case["id_bytes"]))
        s["ws"] = sfg.workspace(sfg.graph_stats_workspace_bytes(case["n"], case["edges"], case["id_bytes"]))
    elif kind == "ensemble":
        s["descs"] = sfg.graph_descs(wl.ensemble_table(case["graphs"], seed=int(seed)))
        s["ws"] = sfg.workspace(sfg.ensemble_workspace_bytes(s["descs"], 1 << 28))
    elif kind == "paths":
        u, v = _rmat(case["n"], case["edges"], seed)
        s["row_ptr"], s["col"] = _simple_csr(case["n"], u, v, _dtype(case["id_bytes"]))
        s["sources"] = np.random.default_rng(int(seed)).integers(0, case["n"], case["sources"])
        s["ws"] = sfg.workspace(sfg.path_stats_workspace_bytes(case["n"]))
    elif kind == "mlp_train":
        g, B = _gen(seed), case["batch"]
        s["shape"] = sfg.mlp_shape(D_IN, case["width"], D_OUT, case["hidden"])
        s["params"] = _params(case, g)
        s["m"] = torch.randn(s["params"].shape, device="cuda", generator=g) * 0.02
        s["v"] = (0.02 + 0.1 * torch.rand(s["params"].shape, device="cuda", generator=g)) ** 2
        rows = 4 * B  # the data set, of which the batch's rows are picked by index
        s["x"] = _features(rows, g)
        s["target"] = torch.randn(rows, D_OUT, device="cuda", generator=g)
        s["mask"] = (torch.rand(rows, D_OUT, device="cuda", generator=g) < 0.9).float()
        s["col_weight"] = 0.5 + torch.rand(D_OUT, device="cuda", generator=g)
        s["rows"] = torch.randperm(rows, device="cuda", generator=g)[:B].contiguous()
        s["lr"] = torch.full((1,), 1e-3, device="cuda")
        s["step"] = torch.full((1,), ADAM_STEP, dtype=torch.int32, device="cuda")
        s["ws"] = sfg.workspace(sfg.mlp_train_workspace_bytes(s["shape"], B))
    elif kind == "mlp_eval":
        g, B = _gen(seed), case["batch"]
        s["shape"] = sfg.mlp_shape(D_IN, case["width"], D_OUT, case["hidden"])
        s["params"] = _params(case, g)
        s["x"] = _features(B, g)
        s["dy"] = torch.zeros(B, D_OUT, device="cuda")
        s["dy"][:, D_OUT - 2] = 1.0
        s["ws"] = sfg.workspace(sfg.mlp_workspace_bytes(s["shape"], B))
    else:
        s["W"] = _seed_matrix(case, seed)
        power = case["edges0"] ** case["k"]
        grown = case["edges0"] * (1 - case["p"]) + (25 - case["edges0"]) * case["p"]  # mean edges of a modified seed
        s["capacity"] = int(1.25 * max(power, case["edges0"] * grown ** (case["k"] - 1))) + 4096
        s["ws"] = sfg.workspace(max(int(sfg.load().kron_perturbed_workspace_bytes(s["capacity"])),
                                    int(sfg.load().kron_xor_random_workspace_bytes(
                                        5, ctypes.c_void_p(s["W"].ctypes.data), case["k"], case["random"], case["id_bytes"]))))
    return s


# ----------------------------------------------------------------------------- run
def _whole(ids, capacity):
    """The array of `capacity` ids that `ids` is the start of, cleared behind it."""
    whole = torch.as_strided(ids, (capacity,), (1,))
    whole[ids.numel():].zero_()
    return whole


def run(state):
    kind, case = state["kind"], state["case"]
    if kind == "kron_csr":
        n0, W = INITIATORS[case["init"]]
        return sfg.kron_generate_csr(n0, W, case["k"], case["edges"], seed=state["seed"], id_bytes=case["id_bytes"],
                                     flags=case["flags"], **state["out"])
    if kind == "pba_csr":
        src, dst = sfg.pba_generate(case["n"], case["m"], case["parts"], case["p"], seed=state["seed"],
                                    id_bytes=case["id_bytes"], src=state["src"], dst=state["dst"], ws=state["ws"])
        return (src, dst) + sfg.edges_to_csr(case["n"], src, dst, flags=sfg.CSR_SYMMETRIZE, row_ptr=state["row_ptr"],
                                             col=state["col"], ws=state["ws"])
    if kind == "csr":
        return sfg.edges_to_csr(case["n"], state["src"], state["dst"], flags=case["flags"], row_ptr=state["row_ptr"],
                                col=state["col"], ws=state["ws"])
    if kind == "stats":
        return sfg.graph_stats(case["n"], state["src"], state["dst"], num_samples=case["samples"], seed=state["seed"],
                               ws=state["ws"])
    if kind == "ensemble":
        return sfg.ensemble_generate(state["descs"], num_samples=case["samples"], stat_seed=5, ws=state["ws"])
    if kind == "paths":
        return sfg.path_stats(case["n"], state["row_ptr"], state["col"], state["sources"], ws=state["ws"])
    if kind == "mlp_train":
        loss = sfg.mlp_train_step(state["shape"], case["batch"], state["params"], state["x"], state["target"], state["m"],
                                  state["v"], state["lr"], state["step"], state["ws"], rows=state["rows"],
                                  mask=state["mask"], col_weight=state["col_weight"])
        return loss, state["params"], state["m"], state["v"]
    if kind == "mlp_eval":
        y = sfg.mlp_forward(state["shape"], state["params"], state["x"], state["ws"])
        _, dx = sfg.mlp_backward(state["shape"], state["params"], state["dy"], state["ws"], want_grad=False, want_dx=True)
        return y, dx
    n = 5 ** case["k"]
    src, dst = sfg.kron_perturbed(5, state["W"], case["k"], case["p"], case["p"], state["capacity"], seed=state["seed"],
                                  id_bytes=case["id_bytes"], ws=state["ws"])
    blocks = sfg.block_matrix(n, src, dst, case["blocks"])
    row_ptr, col = sfg.kron_xor_random(5, state["W"], case["k"], case["random"], seed=state["seed"],
                                       id_bytes=case["id_bytes"], ws=state["ws"])
    # The edge counts depend on the draws; the program keeps its arrays at their capacity, zero beyond the last edge.
    src, dst = _whole(src, state["capacity"]), _whole(dst, state["capacity"])
    col[int(row_ptr[n]):].zero_()
    return src, dst, blocks, row_ptr, col


# ----------------------------------------------------------------------------- work

def work(case):
    """Bytes: inputs read once, outputs written once.  Flops: the matrix products."""
    kind = case["kind"]
    if kind == "kron_csr":
        N = case["edges"] * (2 if case["flags"] & 1 else 1)
        return {"bytes": (2 * case["edges"] + N) * case["id_bytes"] + 8 * (_vertices(case) + 1), "flops": 0}
    if kind == "pba_csr":
        E = case["n"] * case["m"]
        return {"bytes": 4 * E * case["id_bytes"] + 8 * (case["n"] + 1), "flops": 0}
    if kind == "csr":
        N = case["edges"] * (2 if case["flags"] & 1 else 1)
        return {"bytes": (2 * case["edges"] + N) * case["id_bytes"] + 8 * (case["n"] + 1), "flops": 0}
    if kind == "stats":
        return {"bytes": 2 * case["edges"] * case["id_bytes"] + 272, "flops": 0}
    if kind == "ensemble":
        # (no edge list comes back: the tables in, 272 bytes out per graph, and the edges once through memory, which a
        # graph of the recipe's mean size of 1.9 million edges does not avoid)
        return {"bytes": case["graphs"] * (272 + 120 + 2 * 4 * 1.9e6), "flops": 0}
    if kind == "paths":
        groups = (case["sources"] + 63) // 64
        return {"bytes": groups * (2 * case["edges"] * case["id_bytes"] + 8 * case["n"]), "flops": 0}
    if kind in ("mlp_train", "mlp_eval"):
        B = case["batch"]
        params = sum(i * o + o for i, o in _layers(case))
        macs = sum(i * o for i, o in _layers(case))
        if kind == "mlp_train":
            return {"bytes": 4 * (6 * params + B * (D_IN + 2 * D_OUT)) + 8 * B, "flops": 6 * B * macs}
        return {"bytes": 4 * (params + B * (2 * D_IN + 2 * D_OUT)), "flops": 4 * B * macs}
    power = case["edges0"] ** case["k"]
    grown = case["edges0"] * (1 - case["p"]) + (25 - case["edges0"]) * case["p"]
    modified = case["edges0"] * grown ** (case["k"] - 1)
    return {"bytes": case["id_bytes"] * (4 * modified + power + case["random"]) + 8 * (5 ** case["k"] + 1), "flops": 0}


# ----------------------------------------------------------------------------- exact
def _forward(case, params, x):
    """Layers' weights, inputs and pre-activations of the network in float64."""
    p, off, h, keep = params.double(), 0, x.double(), []
    layers = _layers(case)
    for l, (i, o) in enumerate(layers):
        W, b = p[off:off + i * o].reshape(o, i), p[off + i * o:off + i * o + o]
        off += i * o + o
        z = h @ W.t() + b
        keep.append((W, h, z))
        h = z if l == len(layers) - 1 else torch.nn.functional.silu(z)
    return keep, h


def _backward(keep, dy):
    """Gradients of the parameters and of the input, from dy, in float64."""
    grads, d = [], dy
    for l in range(len(keep) - 1, -1, -1):
        W, h, z = keep[l]
        if l < len(keep) - 1:
            s = torch.sigmoid(z)
            d = d * s * (1 + z * (1 - s))
        grads = [(d.t() @ h).reshape(-1), d.sum(0)] + grads
        d = d @ W
    return torch.cat(grads), d


def exact(case, seed):
    """In 64 bits, where an output is a computed number: the surrogate's step and value, and the tail exponent."""
    kind = case["kind"]
    if kind == "mlp_eval":
        s = prepare(case, seed)
        keep, y = _forward(case, s["params"], s["x"])
        return y, _backward(keep, s["dy"].double())[1]
    if kind == "mlp_train":
        s = prepare(case, seed)
        B = case["batch"]
        x, t, w = s["x"][s["rows"]], s["target"][s["rows"]].double(), s["mask"][s["rows"]].double() * s["col_weight"].double()
        keep, y = _forward(case, s["params"], x)
        loss = (w * (y - t) ** 2).sum() / B
        g, _ = _backward(keep, 2 * w * (y - t) / B)
        b1, b2, eps, n = 0.9, 0.999, 1e-8, ADAM_STEP + 1
        m = b1 * s["m"].double() + (1 - b1) * g
        v = b2 * s["v"].double() + (1 - b2) * g * g
        params = s["params"].double() - float(s["lr"]) * (m / (1 - b1 ** n)) / (torch.sqrt(v / (1 - b2 ** n)) + eps)
        return loss.reshape(1), params, m, v
    if kind == "stats":
        u, v = _rmat(case["n"], case["edges"], seed)
        n, E = case["n"], case["edges"]
        deg = torch.bincount(torch.cat([u, v]), minlength=n)
        dmin = 2 * ((2 * E + n - 1) // n)
        tail = deg[deg >= dmin].double()
        gamma = 1 + tail.numel() / torch.log(tail / (dmin - 0.5)).sum() if tail.numel() else torch.tensor(math.nan)
        return None, gamma.reshape(1).double(), None
    return None
