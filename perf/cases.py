"""What the performance of this library is measured on: the calls that a serving program makes while it decodes with
the early-exit predictor, through the public Python entry points, with the buffers such a program keeps between calls
(outputs and workspaces) already allocated.

    listed()            the named cases
    draw(rng)           one more case of the same ranges
    prepare(case, seed) inputs on the GPU, made from the seed alone, and the kept buffers
    run(state)          one pass, returning its outputs
    work(case)          bytes and floating-point operations that a pass cannot do without
    tolerance(case)     how far another correct implementation may be off

Shapes are those of the workloads the benchmark and the tests use (hidden size 4096 / 5120 / 8192, vocabulary 32000 /
128256, K = 4 or 8 speculative tokens, predictor 3K -> 512 -> 1) and odd ones around them.  Distributions as in
paper_2504_08850_amd.synth: LM head ~ N(0, 0.02), RMSNorm weight ~ 1 + N(0, 0.01), hidden states ~ N(0, 1), predictor
weights ~ N(0, 0.05), all fp16; speculative ids uniform or by Zipf(1.1) rank, distinct within a token.
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_2504_08850_amd import specee as sp

EPS, THRESHOLD, H = 1e-5, 0.5, 512


def listed():
    return [
        # One token at one layer, called eagerly: what a decode loop without graphs pays per layer.
        dict(name="predict_one_7b", kind="predict", q4=False, d=4096, V=32000, K=4, B=1, ids="uniform"),
        # Batched decode of 16 sequences over a 40-layer model: one dependent predictor call per layer, captured once in
        # a graph and replayed for every token position.
        dict(name="decode_graph_13b", kind="graph", d=5120, V=32000, K=4, B=16, L=40, ids="zipf"),
        # Many independent tokens at one layer (large serving batch, or predictor training data): bound by row gathers.
        dict(name="predict_batch_7b", kind="predict", q4=False, d=4096, V=32000, K=4, B=2043, ids="uniform"),
        # The same on the 4-bit group-quantised head.
        dict(name="predict_q4_batch_7b", kind="predict", q4=True, group=128, d=4096, V=32000, K=4, B=8000, ids="uniform"),
        # One token tree (60 nodes): one speculative-decoding step of one sequence at one layer.
        dict(name="tree_one_7b", kind="tree", q4=False, d=4096, V=32000, K=4, N=60, G=1, Mcap=64),
        # 64 sequences decode speculatively together.
        dict(name="trees_64_7b", kind="tree", q4=False, d=4096, V=32000, K=4, N=60, G=64, Mcap=64),
        # The large-vocabulary tree shape in the largest batch that the benchmark runs.
        dict(name="trees_256_large_vocab", kind="tree", q4=False, d=8192, V=128256, K=8, N=64, G=256, Mcap=256),
        # 16 sequences decode speculatively on the quantised head.
        dict(name="trees_q4_16_7b", kind="tree", q4=True, group=128, d=4096, V=32000, K=4, N=60, G=16, Mcap=64),
        # Verification of one token after a positive prediction: one pass over the whole head.
        dict(name="verify_one_7b", kind="verify", q4=False, d=4096, V=32000, K=4, N=1, gated=False),
        # Verification of a batch of 16 sequences on the quantised head.
        dict(name="verify_q4_16_7b", kind="verify", q4=True, group=128, d=4096, V=32000, K=4, N=16, gated=False),
        # The full head for the 64 nodes of a tree, large vocabulary: the search space that the predictor replaces.
        dict(name="head_64_large_vocab", kind="head", q4=False, d=8192, V=128256, N=64),
        # One token down a 32-layer stack in one call, under the online scheduler's active set: predictors until one
        # fires, verification, exit (usually in the last third of the stack).
        dict(name="layer_loop_7b", kind="loop", q4=False, d=4096, V=32000, K=4, L=32, B=1),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """The kinds and ranges of the listed cases; a draw never costs more than the largest of them."""
    kind = rng.choice(["predict", "predict", "graph", "tree", "tree", "verify", "head", "loop"])
    q4 = rng.random() < 0.4
    d, V = rng.choice([(4096, 32000), (5120, 32000), (4096, 32000), (2048, 50280), (3072, 32003), (4608, 24001)])
    if not q4 and rng.random() < 0.2:
        d, V = rng.choice([(3080, 32001), (4104, 20011)])  # rows that are not a whole number of 128-byte lines
    K = rng.choice([4, 4, 4, 3, 5, 8])
    group = rng.choice([128, 128, 64])
    if kind == "predict":
        c = dict(kind=kind, q4=q4, d=d, V=V, K=K, B=_log(rng, 1, 8000), ids=rng.choice(["uniform", "zipf"]))
    elif kind == "graph":
        q4 = False
        c = dict(kind=kind, d=d, V=V, K=K, B=_log(rng, 1, 24), L=rng.randint(16, 40), ids=rng.choice(["uniform", "zipf"]))
    elif kind == "tree":
        if not q4 and rng.random() < 0.3:
            d, V, K = 8192, 128256, 8
            N, Mcap, G = rng.randint(40, 64), 256, _log(rng, 1, 128)
        else:
            N, Mcap, G = rng.randint(8, 64), 64, _log(rng, 1, 128)
        c = dict(kind=kind, q4=q4, d=d, V=V, K=K, N=N, G=G, Mcap=Mcap)
    elif kind == "verify":
        c = dict(kind=kind, q4=q4, d=d, V=V, K=K, N=_log(rng, 1, 16 if q4 else 64), gated=rng.random() < 0.3)
    elif kind == "head":
        if not q4 and rng.random() < 0.3:
            d, V = 8192, 128256
        c = dict(kind=kind, q4=q4, d=d, V=V, N=_log(rng, 1, 16 if q4 else 64))
    else:
        c = dict(kind=kind, q4=q4, d=d, V=V, K=K, L=rng.randint(24, 40), B=_log(rng, 1, 4))
    if q4:
        c["group"] = group
    return c


# ---- inputs -------------------------------------------------------------------------------------------------------

def _ids(case, seed, n, pool):
    """[n][K] int32: K distinct ids per row, uniform or by Zipf(1.1) rank over `pool` random tokens (None: all V)."""
    rng = np.random.Generator(np.random.PCG64([int(seed), 6]))
    V, K = case["V"], case["K"]
    zipf = pool is not None or case.get("ids") == "zipf"
    size = V if pool is None else pool
    table = rng.permutation(V)[:size].astype(np.int32)
    cdf = np.cumsum(np.arange(1, size + 1, dtype=np.float64) ** -1.1) if zipf else None

    def some(m):
        if cdf is None:
            return rng.integers(0, size, m)
        return np.minimum(np.searchsorted(cdf, rng.random(m) * cdf[-1]), size - 1)

    out = np.empty((n, K), dtype=np.int64)
    for k in range(K):  # successive sampling without replacement: redraw what a row already holds
        out[:, k] = some(n)
        while k:
            bad = np.nonzero((out[:, :k] == out[:, k:k + 1]).any(axis=1))[0]
            if not bad.size:
                break
            out[bad, k] = some(bad.size)
    return table[out]


def _tree_ids(case, seed):
    G, N, K = case["G"], case["N"], case["K"]
    pool = max(K, min(case["Mcap"], case["V"]))
    return np.stack([_ids(case, seed * 1009 + g, N, pool) for g in range(G)])


class _Draw:
    def __init__(self, seed):
        self.g = torch.Generator(device="cuda")
        self.g.manual_seed(int(seed))

    def normal(self, shape, std=1.0, mean=0.0):
        t = torch.empty(shape, dtype=torch.float16, device="cuda")
        return t.normal_(mean, std, generator=self.g)

    def probs(self, shape):
        e = torch.empty(shape, dtype=torch.float32, device="cuda").exponential_(generator=self.g)
        return e / e.sum(-1, keepdim=True)

    def mlp(self, K, lead=()):
        return dict(W1=self.normal(lead + (H, 3 * K), 0.05), w2=self.normal(lead + (H,), 0.05))

    def q4_head(self, V, d, group):
        """A head ~ N(0, 0.02), quantised with plain asymmetric min/max rounding per group."""
        ng = d // group
        q = torch.empty((V, d // 8), dtype=torch.int32, device="cuda")
        scales = torch.empty((V, ng), dtype=torch.float16, device="cuda")
        zeros = torch.empty_like(scales)
        shifts = (4 * torch.arange(8, device="cuda", dtype=torch.int32))
        for r in range(0, V, 16384):
            w = self.normal((min(16384, V - r), ng, group), 0.02).float()
            lo, hi = w.amin(2), w.amax(2)
            s = ((hi - lo) / 15.0).half()
            z = torch.round(-lo / s.float()).clamp_(0, 15)
            code = torch.round(w / s.float()[:, :, None] + z[:, :, None]).clamp_(0, 15).to(torch.int32)
            q[r:r + w.shape[0]] = (code.view(-1, d // 8, 8) << shifts).sum(2, dtype=torch.int32)
            scales[r:r + w.shape[0]] = s
            zeros[r:r + w.shape[0]] = z.half()
        return dict(qweight=q, scales=scales, zeros=zeros, group=group)


def _f32(*shape):
    return torch.zeros(shape, dtype=torch.float32, device="cuda")


def _i32(*shape):
    return torch.zeros(shape, dtype=torch.int32, device="cuda")


def _workspace(op, case, n, Mcap=0):
    dims = sp.Dims(case["d"], case["V"], case.get("K", 1), H, EPS, THRESHOLD)
    return torch.empty(max(16, sp.workspace_bytes(op, dims, n, Mcap)), dtype=torch.uint8, device="cuda")


def _predict_out(B, K):
    return dict(logits=_f32(B, K), probs=_f32(B, K), scores=_f32(B), exit=_i32(B))


def prepare(case, seed):
    kind, d, V = case["kind"], case["d"], case["V"]
    K, q4 = case.get("K", 1), case.get("q4", False)
    dr = _Draw(seed)
    head = dr.q4_head(V, d, case["group"]) if q4 else dict(lm_head=dr.normal((V, d), 0.02))
    gamma = dr.normal((d,), 0.01, 1.0)
    s = dict(kind=kind, q4=q4)
    if kind == "predict":
        B = case["B"]
        s["args"] = dict(hidden=dr.normal((B, d)), gamma=gamma, ids=torch.from_numpy(_ids(case, seed, B, None)).cuda(),
                         prev_probs=dr.probs((B, K)), out=_predict_out(B, K), **head, **dr.mlp(K))
    elif kind == "graph":
        B, L = case["B"], case["L"]
        ids = torch.from_numpy(_ids(case, seed, B, None)).cuda()
        hidden, mlp = dr.normal((L, B, d)), dr.mlp(K, (L,))
        prev = _f32(B, K)
        every = dict(logits=_f32(L, B, K), probs=_f32(L, B, K), scores=_f32(L, B), exit=_i32(L, B))
        outs = [{k: v[l] for k, v in every.items()} for l in range(L)]

        def chain():
            p = prev
            for l in range(L):
                sp.predict(hidden[l], gamma, head["lm_head"], ids, p, mlp["W1"][l], mlp["w2"][l], out=outs[l])
                p = outs[l]["probs"]

        chain()  # first launches outside the capture
        torch.cuda.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph):
            chain()
        s.update(graph=graph, outs=every, keep=(hidden, gamma, head, ids, prev, mlp))
    elif kind == "tree":
        G, N, Mcap = case["G"], case["N"], case["Mcap"]
        cuts = np.round(N * np.cumsum([0, 4, 8, 12, 14, 12, 10]) / 60.0).astype(int)  # nodes per level, 60-node tree
        rng = np.random.Generator(np.random.PCG64([int(seed), 10]))
        parent = np.full((G, N), -1, dtype=np.int32)
        for l in range(1, 6):
            a, b, e = cuts[l - 1], cuts[l], cuts[l + 1]
            if b > a:
                parent[:, b:e] = rng.integers(a, b, (G, e - b))
        out = dict(merged=_i32(G, Mcap), M=_i32(G), cols=_i32(G, N, K), logits=_f32(G, N, K), probs=_f32(G, N, K),
                   scores=_f32(G, N), exit=_i32(G, N), path_exit=_i32(G, N))
        s["args"] = dict(hidden=dr.normal((G, N, d)), gamma=gamma, ids=torch.from_numpy(_tree_ids(case, seed)).cuda(),
                         prev_probs=dr.probs((G, N, K)), parent=torch.from_numpy(parent).cuda(), Mcap=Mcap, out=out,
                         **head, **dr.mlp(K))
        if not q4:
            s["args"]["workspace"] = _workspace(sp.OP_PREDICT_TREE, case, G * N, Mcap)
    elif kind in ("verify", "head"):
        N = case["N"]
        s["args"] = dict(hidden=dr.normal((N, d)), gamma=gamma, **head)
        if kind == "verify":
            op = sp.OP_VERIFY_Q4 if q4 else sp.OP_VERIFY
            s["args"].update(ids=torch.from_numpy(_ids(case, seed, N, None)).cuda(), workspace=_workspace(op, case, N),
                             out=dict(token=_i32(N), max_logit=_f32(N), hit=_i32(N)))
            if case["gated"]:  # as the predictor's exit flags: about half of the batch is verified
                gate = torch.rand((N,), generator=dr.g, device="cuda") < 0.5
                gate[0] = True
                s["args"]["gate"] = gate.to(torch.int32)
        else:
            s["args"]["out"] = _f32(N, V)
    else:  # loop
        s["args"] = _loop_args(case, seed, dr, head, gamma)
    return s


def _loop_args(case, seed, dr, head, gamma):
    """Hidden states drift down the stack and turn towards one of the token's speculative rows before its exit layer;
    the predictors read the largest local probability, so they fire about there and the verification then accepts."""
    L, B, K, d, V = case["L"], case["B"], case["K"], case["d"], case["V"]
    rng = np.random.Generator(np.random.PCG64([int(seed), 12]))
    ids_np = _ids(case, seed, B, None)
    ids = torch.from_numpy(ids_np).cuda()
    exits = rng.integers(2 * L // 3, L - 2, B)
    if case["q4"]:
        rows = torch.empty((B, d), device="cuda")
        shifts = 4 * torch.arange(8, device="cuda", dtype=torch.int32)
        for b in range(B):
            v = int(ids_np[b, 0])
            code = ((head["qweight"][v][:, None] >> shifts) & 15).reshape(-1, case["group"]).float()
            rows[b] = (head["scales"][v].float()[:, None] * (code - head["zeros"][v].float()[:, None])).reshape(-1)
    else:
        rows = head["lm_head"][ids[:, 0].long()].float()
    rows = rows * (12.0 / rows.square().sum(1, keepdim=True))  # adds 12 to the row's own logit, well above the others
    hidden = torch.empty((L, B, d), dtype=torch.float16, device="cuda")
    cur = dr.normal((B, d)).float()
    for l in range(L):
        cur = cur + 0.1 * dr.normal((B, d)).float() if l else cur
        pull = np.clip((l - exits + 3) / 3.0, 0.0, 1.0).astype(np.float32)
        hidden[l] = (cur / cur.square().mean(1, keepdim=True).sqrt() + torch.from_numpy(pull).cuda()[:, None] * rows).half()
    mlp = dr.mlp(K, (L,))
    for k in range(K):  # hidden unit k: relu(p_k - 0.9), weighted so that the score passes 1/2 at p_k = 0.95
        mlp["W1"][:, k] = 0
        mlp["W1"][:, k, K + k] = 1.0
        mlp["w2"][:, k] = 100.0
    mlp["b1"] = torch.zeros((L, H), dtype=torch.float16, device="cuda")
    mlp["b1"][:, :K] = -0.9
    mlp["b2"] = torch.full((L,), -5.0, dtype=torch.float16, device="cuda")
    # active layers: every eighth, and the neighbourhood of the recent exits (here: of these tokens' own)
    active = np.zeros(L, dtype=np.int32)
    active[::8] = 1
    for e in exits:
        active[max(0, e - 3):e + 3] = 1
    out = dict(logits=_f32(L, B, K), probs=_f32(L, B, K), scores=_f32(L, B), exit=_i32(L, B), ver_token=_i32(L, B),
               hit=_i32(L, B), exit_layer=_i32(B), token=_i32(B), status=_i32(B))
    return dict(hidden=hidden, gamma=gamma, ids=ids, active=torch.from_numpy(active).cuda(), out=out,
                workspace=_workspace(sp.OP_LAYER_LOOP, case, B), **head, **mlp)


# ---- one pass -----------------------------------------------------------------------------------------------------

_CALLS = {("predict", False): sp.predict, ("predict", True): sp.predict_q4, ("tree", False): sp.predict_tree,
          ("tree", True): sp.predict_tree_q4, ("verify", False): sp.verify, ("verify", True): sp.verify_q4,
          ("head", False): sp.lm_head_gemv, ("head", True): sp.lm_head_gemv_q4, ("loop", False): sp.layer_loop,
          ("loop", True): sp.layer_loop_q4}


def run(state):
    if state["kind"] == "graph":
        state["graph"].replay()
        return state["outs"]
    out = _CALLS[state["kind"], state["q4"]](eps=EPS, **({} if state["kind"] in ("verify", "head") else
                                                         {"threshold": THRESHOLD}), **state["args"])
    if isinstance(out, dict) and "_workspace" in out:
        return {k: v for k, v in out.items() if k != "_workspace"}
    return out


# ---- what a pass cannot do without ----------------------------------------------------------------------------------

def work(case):
    kind, d, V = case["kind"], case["d"], case["V"]
    K, L = case.get("K", 1), case.get("L", 1)
    row = d // 2 + 4 * d // case["group"] if case.get("q4") else 2 * d
    mlp = 2 * (3 * K * H + H)
    per_token = 4 * (K + K + 2 * K + 2)  # ids, previous probabilities, logits, probabilities, score, exit flag
    mlp_flops = 2 * (3 * K * H + H)
    if kind in ("predict", "graph"):
        B = case["B"]
        rows = len(np.unique(_ids(case, 0, B, None)))
        return dict(bytes=L * (B * 2 * d + mlp + B * per_token) + 2 * d + rows * row,
                    flops=L * B * (2 * K * d + 2 * d + mlp_flops))
    if kind == "tree":
        G, N = case["G"], case["N"]
        ids = _tree_ids(case, 0)
        merged = sum(len(np.unique(t)) for t in ids)
        return dict(bytes=G * N * 2 * d + 2 * d + len(np.unique(ids)) * row + mlp +
                    G * (N * (per_token + 4 * K + 8) + 4 * case["Mcap"] + 4),
                    flops=2 * N * merged * d + G * N * (2 * d + mlp_flops))
    if kind in ("verify", "head"):
        N = case["N"]
        outputs = 4 * N * V if kind == "head" else N * (4 * K + 12)
        return dict(bytes=V * row + N * 2 * d + 2 * d + outputs, flops=2 * N * V * d + 2 * N * d)
    # loop: about half of the stack's layers are evaluated before the exit, and one verification is made per token
    B, evaluated = case["B"], min(L, 4 + 5)
    return dict(bytes=evaluated * (B * 2 * d + mlp) + 2 * d + B * K * row + V * row +
                L * B * 4 * (2 * K + 4) + B * (4 * K + 12),
                flops=evaluated * B * (2 * K * d + 2 * d + mlp_flops) + 2 * B * V * d)


def tolerance(case):
    """fp16 inputs, fp32 products and sums.  Measured against float64 over the listed cases: logits are off by 0.5e-7 to
    8e-7 (2-norm) and at most 6.4e-6 of their root mean square, probabilities and scores by less; four times that is
    stated.  An exit flag may flip where a score lies within such a distance of the threshold."""
    return {"rel": 3e-6, "max": 3e-5, "differ": 1e-3}
