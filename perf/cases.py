"""The work a program does through this framework's entry points, as cases to be timed and compared.

Kinds of case:
  minibatch  what every training step begins with: uniform sample, induced CSR, labels (and features) of the sample;
             with shard > 1 one tile of a shard x shard partition of the matrix, and its transpose
  layer      one GCN layer, forward and backward: an input layer reads all features through the sample, a hidden one
             the activations of the layer below, whose ReLU mask it applies to the gradient it hands down
  head       the classifier layer: forward, cross-entropy and its gradient, backward
  block      one residual block of the complete model (aggregate, transform, RMSNorm + ReLU + dropout + skip) and
             its backward pass
  eval       the full-graph forward pass of a trained stack
  step       whole training steps of a stack (GcnStep): one alone, or a run of steps that overlap
Sizes follow the five workload configurations of this repository (4 k to 111 M vertices, samples of 1 k to 2^20,
widths 32 to 608) and ragged neighbours of them.  Graphs are R-MAT (a, b, c, d = .57, .19, .19, .05) with relabelled
vertices, features and gradients are normal, hidden activations are the positive part of normals.
"""
import math

import torch

import paper_2604_02651_amd as sg

DEV = "cuda:0"
M32 = 0xFFFFFFFF


def listed():
    return [
        # the smallest training step (4 k vertices, fp32), issued call by call: launches and latency
        dict(name="step_small_fp32", kind="step", N=4096, edges=32768, rows=1024, dims="32-64-8", bf16=False, steps=1, logits=True),
        # four overlapped steps on a co-purchase-sized graph, bfloat16 operands and storage, as a training loop runs them
        dict(name="steps_large_bf16", kind="step", N=2449029, edges=61859140, rows=262144, dims="100-256-256-47", bf16=True, steps=4,
             logits=True),
        # mini-batch construction on a small graph (int32 offsets), where launches weigh most
        dict(name="minibatch_medium", kind="minibatch", N=262144, edges=2097152, rows=32768, i64=False, feat=0, shard=1),
        # the same on a co-purchase-sized graph: 13 M edges of sampled rows are tested
        dict(name="minibatch_large", kind="minibatch", N=2449029, edges=61859140, rows=262144, i64=True, feat=0, shard=1),
        # a sparse sample (2.5 %) of a citation-sized graph of tens of millions of vertices, odd sizes
        dict(name="minibatch_sparse", kind="minibatch", N=40000003, edges=100000000, rows=999983, i64=True, feat=0, shard=1),
        # hidden layer of a mini-batch of the medium graph in fp32: 2.9 entries a row
        dict(name="layer_medium_fp32", kind="layer", rows=32768, deg=2.9, d_in=256, d_out=256, bf16=False, first=False, xform=False),
        # input layer on a social-network-shaped mini-batch in fp32: 140 entries a row, 608 (padded 602) features
        dict(name="layer_dense_fp32", kind="layer", rows=65536, deg=140.0, d_in=608, d_out=256, bf16=False, first=True, xform=True),
        # hidden layer with bfloat16 operands and storage, 2^18 rows of 6.4 entries
        dict(name="layer_large_bf16", kind="layer", rows=262144, deg=6.4, d_in=256, d_out=256, bf16=True, first=False, xform=False),
        # hidden layer of the largest mini-batch: 2^20 rows of 1.3 entries
        dict(name="layer_xlarge_bf16", kind="layer", rows=1048576, deg=1.27, d_in=256, d_out=256, bf16=True, first=False, xform=False),
        # classifier layer and loss of the largest mini-batch, 172 classes, no logits kept
        dict(name="head_xlarge_bf16", kind="head", rows=1048576, deg=1.27, d_in=256, d_out=172, bf16=True, fused=True, logits=False),
        # a block of the complete model at ragged sizes in fp32 with dropout
        dict(name="block_ragged_fp32", kind="block", rows=30011, deg=3.9, d=200, bf16=False, drop=0.1),
        # evaluation: the forward pass over all vertices of a graph with 51 entries a row
        dict(name="eval_graph", kind="eval", N=600011, edges=15000000, dims="100-256-47", bf16=True),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["minibatch", "minibatch", "layer", "layer", "layer", "layer", "head", "head", "block", "eval", "step"])
    bf16 = rng.random() < 0.5
    if kind == "minibatch":
        N = _log(rng, 3000, 8000000)
        rows = _log(rng, max(500, N // 60), N // 3)
        edges = min(int(N * _log(rng, 2, 200) / 2), 40000000, N * 100)
        return dict(kind=kind, N=N, edges=edges, rows=rows, i64=rng.random() < 0.5, feat=rng.choice([0, 0, rng.randint(5, 130)]),
                    shard=rng.choice([1, 1, 2, 3]))
    if kind == "eval":
        N = _log(rng, 5000, 500000)
        return dict(kind=kind, N=N, edges=int(N * rng.uniform(2, 25)), dims="%d-%d-%d" % (rng.randint(20, 130), rng.randint(33, 256),
                                                                                          rng.randint(5, 64)), bf16=bf16)
    if kind == "step":
        N = _log(rng, 4000, 400000)
        return dict(kind=kind, N=N, edges=N * rng.randint(4, 40), rows=_log(rng, 1000, N // 4 + 1), steps=rng.choice([1, 2, 4]), bf16=bf16,
                    dims="%d-%d-%d-%d" % (rng.randint(20, 100), h := rng.choice([64, 100, 128, 200, 256]), h, rng.randint(5, 60)),
                    logits=rng.random() < 0.5)
    rows = _log(rng, 700, 900000 if bf16 else 200000)
    deg = round(math.exp(rng.uniform(math.log(1.2), math.log(min(150.0, 6e6 / rows, rows / 20)))), 2)
    if kind == "block":
        return dict(kind=kind, rows=min(rows, 200000), deg=deg, d=rng.choice([64, 128, 256, rng.randint(24, 300)]), bf16=bf16,
                    drop=rng.choice([0.0, 0.1, 0.5]))
    d_in, d_out = (rng.choice([32, 64, 100, 128, 256, 256, rng.randint(17, 320)]) for _ in range(2))
    if kind == "head":
        return dict(kind=kind, rows=rows, deg=deg, d_in=d_in, d_out=rng.choice([rng.randint(3, 64), rng.randint(40, 200)]), bf16=bf16,
                    fused=rng.random() < 0.5, logits=rng.random() < 0.5)
    first = rng.random() < 0.4
    if first and not bf16 and rows < 100000 and rng.random() < 0.3:
        d_in = rng.choice([602, 608, rng.randint(321, 640)])
    return dict(kind=kind, rows=rows, deg=deg, d_in=d_in, d_out=d_out, bf16=bf16, first=first, xform=d_out < d_in)


# ---------------------------------------------------------------------------------------------- inputs

def _gen(seed, k):
    return torch.Generator(device=DEV).manual_seed((seed * 1000003 + k * 7919 + 17) & 0x7FFFFFFFFFFF)


def _edges(N, count, gen):
    """`count` distinct undirected R-MAT edges (as lo * N + hi), vertices relabelled at random; fewer where they repeat too often."""
    scale = max(1, (N - 1).bit_length())
    perm = torch.randperm(N, device=DEV, generator=gen)
    keys = torch.empty(0, dtype=torch.int64, device=DEV)
    for _ in range(12):
        need = count - keys.numel()
        if need <= 0:
            break
        n = min(1 << 25, max(4096, int(1.7 * need)))
        u = torch.zeros(n, dtype=torch.int64, device=DEV)
        v = torch.zeros(n, dtype=torch.int64, device=DEV)
        for _ in range(scale):
            r = torch.rand(n, device=DEV, generator=gen)
            u = (u << 1) | (r >= 0.76)
            v = (v << 1) | (((r >= 0.57) & (r < 0.76)) | (r >= 0.95))
        ok = (u < N) & (v < N) & (u != v)
        u, v = perm[u[ok]], perm[v[ok]]
        keys = torch.unique(torch.cat([keys, torch.minimum(u, v) * N + torch.maximum(u, v)]))
    if keys.numel() > count:
        keys = keys[torch.randperm(keys.numel(), device=DEV, generator=gen)[:count]]
    return keys


def _graph(N, edges, gen):
    """Canonical CSR of A + I: rowptr int64, colidx int32."""
    keys = _edges(N, edges, gen)
    lo, hi = keys // N, keys % N
    loops = torch.arange(N, device=DEV)
    keys = torch.sort(torch.cat([keys, hi * N + lo, loops * N + loops]))[0]
    del lo, hi
    rowptr = torch.zeros(N + 1, dtype=torch.int64, device=DEV)
    rowptr[1:] = torch.cumsum(torch.bincount(keys // N, minlength=N), 0)
    return rowptr, (keys % N).to(torch.int32)


def _matrix(case, gen):
    """A normalised mini-batch matrix of about rows * deg entries: rowptr, colidx, val (rescaled as if one vertex in eight were sampled)."""
    B = case["rows"]
    rowptr, colidx = _graph(B, int(B * (case["deg"] - 1) / 2), gen)
    deg = (rowptr[1:] - rowptr[:-1]).double()
    row = torch.repeat_interleave(torch.arange(B, device=DEV), rowptr[1:] - rowptr[:-1])
    val = torch.rsqrt(deg[row] * deg[colidx.long()]) * torch.where(row == colidx, 1.0, 8.0)
    return rowptr.to(torch.int32), colidx, val.float()


def _csr(ctx, B, rowptr, colidx, val):
    nnz = colidx.numel()
    A = sg.Csr(B, B, 2 * nnz + 16 * B + 65536, DEV)
    A.rowptr.copy_(rowptr)
    A.colidx[:nnz] = colidx
    A.val[:nnz] = val
    A.nnz_dev.fill_(nnz)
    sg.sgnn_csr_plan(ctx, A)
    return A


def _mat(rows, d, dtype):
    """rows x d with every row on a 64-byte boundary."""
    pad = 32 if dtype == torch.bfloat16 else 16
    return torch.empty((rows, (d + pad - 1) // pad * pad), dtype=dtype, device=DEV)[:, :d]


def _normal(rows, d, gen, dtype=torch.float32, relu=False, scale=1.0):
    m = _mat(rows, d, dtype)
    for r0 in range(0, rows, 1 << 18):
        x = torch.randn((min(1 << 18, rows - r0), d), device=DEV, generator=gen) * scale
        m[r0:r0 + x.shape[0]] = x.relu_() if relu else x
    return m


def _glorot(a, b, gen):
    return (torch.rand((a, b), device=DEV, generator=gen) * 2 - 1) * math.sqrt(6.0 / (a + b))


def _bias(d, gen):
    return torch.rand(d, device=DEV, generator=gen) * 0.2 - 0.1


def _dims(case):
    return [int(x) for x in case["dims"].split("-")]


def prepare(case, seed):
    return globals()["_prepare_" + case["kind"]](case, seed)


def run(state):
    return state["run"](state)


def _inputs_minibatch(case, seed):
    N, gen = case["N"], _gen(seed, 1)
    rowptr, colidx = _graph(N, case["edges"], gen)
    labels = torch.randint(0, 47, (N,), device=DEV, dtype=torch.int32, generator=gen)
    X = torch.randn((N, case["feat"]), device=DEV, generator=gen) if case["feat"] else None
    return rowptr, colidx, labels, X


def _capacity(N, E, B):
    return int(min(E, 2 * (B + (E - N) * (B / N) * ((B - 1) / max(N - 1, 1))) + 16 * B + 65536))


def _tile(case):
    """The vertex ranges of the tile: the second block of rows, the first of columns (all of both without a partition)."""
    N, g = case["N"], case["shard"]
    return (0, N, 0, N) if g == 1 else (N // g, 2 * N // g, 0, N // g)


def _prepare_minibatch(case, seed):
    N, B = case["N"], case["rows"]
    rowptr, colidx, labels, X = _inputs_minibatch(case, seed)
    E = colidx.numel()
    ctx = sg.Context(0)
    cap = _capacity(N, E, B)
    ctx.reserve(N, E, B, 256, cap)
    W = (N + 63) // 64
    i32 = dict(dtype=torch.int32, device=DEV)
    return dict(run=_run_minibatch, case=case, seed=seed, ctx=ctx, rowptr=rowptr if case["i64"] else rowptr.to(torch.int32), colidx=colidx,
                labels=labels, X=X, S=torch.empty(B, **i32), bitmap=torch.empty(W, dtype=torch.int64, device=DEV),
                rank=torch.empty(W, **i32), A=sg.Csr(B, B, cap, DEV), At=sg.Csr(B, B, cap, DEV) if case["shard"] > 1 else None,
                y=torch.empty(B, **i32), X_S=torch.empty((B, case["feat"]), device=DEV) if X is not None else None)


def _run_minibatch(s):
    c, ctx, A, At = s["case"], s["ctx"], s["A"], s["At"]
    N, B = c["N"], c["rows"]
    sg.sgnn_sample_uniform(ctx, N, B, s["seed"], s["seed"] & 255, s["S"], s["bitmap"], s["rank"])
    if At is None:
        sg.sgnn_induced_csr(ctx, N, s["rowptr"], s["colidx"], None, s["S"], B, s["bitmap"], s["rank"], A)
    else:
        sg.sgnn_induced_csr_range(ctx, N, s["rowptr"], s["colidx"], None, s["S"], B, s["bitmap"], s["rank"], *_tile(c), A)
        sg.sgnn_csr_transpose(ctx, A, At)
    sg.sgnn_gather_rows(ctx, s["X"], s["S"], B, s["X_S"], s["labels"], s["y"])
    out = dict(S=s["S"], bitmap=s["bitmap"], rank=s["rank"], rowptr=A.rowptr, colidx=A.colidx, val=A.val, nnz=A.nnz_dev, y=s["y"])
    if At is not None:
        out.update(t_rowptr=At.rowptr, t_colidx=At.colidx, t_val=At.val)
    if s["X_S"] is not None:
        out["X_S"] = s["X_S"]
    return out


def _inputs_layer(case, seed):
    """Everything the layer's two calls read, in the storage a bfloat16 or fp32 stack keeps it in."""
    B, d_in, d_out, gen = case["rows"], case["d_in"], case["d_out"], _gen(seed, 2)
    act = torch.bfloat16 if case["bf16"] else torch.float32
    A = _matrix(case, gen)
    if case["first"]:
        S = torch.sort(torch.randperm(2 * B, device=DEV, generator=gen)[:B])[0].to(torch.int32)
        H = _normal(2 * B, d_in, gen, torch.float32 if case["xform"] else act)
    else:
        S, H = None, _normal(B, d_in, gen, act, relu=True)
    # the gradient from the layer above, already masked by this layer's ReLU there
    dY = _normal(B, d_out, gen, torch.float32 if case["xform"] else act, scale=1.0 / B)
    dY *= torch.rand((B, d_out), device=DEV, generator=gen) < 0.5
    return A, S, H, _glorot(d_in, d_out, gen), _bias(d_out, gen), dY


def _prepare_layer(case, seed):
    B, d_in, d_out = case["rows"], case["d_in"], case["d_out"]
    (rowptr, colidx, val), S, H, W, b, dY = _inputs_layer(case, seed)
    act = torch.bfloat16 if case["bf16"] else torch.float32
    ctx = sg.Context(0)
    ctx.reserve(2 * B, colidx.numel(), B, max(d_in, d_out), 2 * colidx.numel() + 16 * B + 65536)
    return dict(run=_run_layer, case=case, ctx=ctx, A=_csr(ctx, B, rowptr, colidx, val), S=S, H=H, W=W, b=b, dY=dY, Y=_mat(B, d_out, act),
                T=None if case["xform"] else _mat(B, d_in, act), dH=None if case["first"] else _mat(B, d_in, act),
                dW=torch.empty_like(W), db=torch.empty_like(b))


def _run_layer(s):
    c, ctx, A, S, H = s["case"], s["ctx"], s["A"], s["S"], s["H"]
    flags = sg.SGNN_RELU | (sg.SGNN_BF16_MFMA if c["bf16"] else 0) | (sg.SGNN_XFORM_FIRST if c["xform"] else 0)
    sg.sgnn_gcn_fwd(ctx, A, H, s["W"], s["b"], flags, s["Y"], s["T"], row_index=S)
    saved = H if c["xform"] else s["T"]
    sg.sgnn_gcn_bwd(ctx, A, saved, s["W"], s["Y"], s["dY"], flags | sg.SGNN_DY_MASKED, s["dH"], s["dW"], s["db"],
                    row_index=S if c["xform"] else None, H_in=None if c["first"] else H)
    out = dict(Y=s["Y"], dW=s["dW"], db=s["db"])
    if not c["xform"]:
        out["T"] = s["T"]
    if not c["first"]:
        out["dH"] = s["dH"]
    return out


def _inputs_head(case, seed):
    B, gen = case["rows"], _gen(seed, 3)
    A = _matrix(case, gen)
    H = _normal(B, case["d_in"], gen, torch.bfloat16 if case["bf16"] else torch.float32, relu=True)
    y = torch.randint(0, case["d_out"], (B,), device=DEV, dtype=torch.int32, generator=gen)
    return A, H, _glorot(case["d_in"], case["d_out"], gen), _bias(case["d_out"], gen), y


def _prepare_head(case, seed):
    B, d_in, C = case["rows"], case["d_in"], case["d_out"]
    (rowptr, colidx, val), H, W, b, y = _inputs_head(case, seed)
    act = torch.bfloat16 if case["bf16"] else torch.float32
    ctx = sg.Context(0)
    ctx.reserve(B, colidx.numel(), B, max(d_in, C), 2 * colidx.numel() + 16 * B + 65536)
    xform = C < d_in
    fused = xform and case["fused"]
    return dict(run=_run_head, case=case, fused=fused, xform=xform, ctx=ctx, A=_csr(ctx, B, rowptr, colidx, val), H=H, W=W, b=b, y=y,
                P=_mat(B, C, act) if fused else None, T=None if xform else _mat(B, d_in, act),
                O=None if fused and not case["logits"] else _mat(B, C, torch.float32), loss=torch.zeros(1, device=DEV), dO=_mat(B, C, act),
                dH=_mat(B, d_in, act), dW=torch.empty_like(W), db=torch.empty_like(b))


def _run_head(s):
    ctx, A, H, W, O = s["ctx"], s["A"], s["H"], s["W"], s["O"]
    mfma = sg.SGNN_BF16_MFMA if s["case"]["bf16"] else 0
    flags = mfma | (sg.SGNN_XFORM_FIRST if s["xform"] else 0)
    if s["fused"]:
        sg.sgnn_gemm(ctx, False, False, H, W, None, mfma, s["P"])
        sg.sgnn_spmm_xent(ctx, A, s["P"], s["b"], s["y"], s["loss"], s["dO"], O=O, dO_colsum=s["db"])
    else:
        sg.sgnn_gcn_fwd(ctx, A, H, W, s["b"], flags, O, s["T"])
        sg.sgnn_softmax_xent(ctx, O, s["y"], s["loss"], s["dO"], dO_colsum=s["db"])
    sg.sgnn_gcn_bwd(ctx, A, H if s["xform"] else s["T"], W, None, s["dO"], flags, s["dH"], s["dW"], None, H_in=H)
    out = dict(loss=s["loss"], dO=s["dO"], db=s["db"], dH=s["dH"], dW=s["dW"])
    if O is not None:
        out["O"] = O
    return out


EPS = 1e-6


def _inputs_block(case, seed):
    B, d, gen = case["rows"], case["d"], _gen(seed, 4)
    A = _matrix(case, gen)
    X, dY, Z = _normal(B, d, gen), _normal(B, d, gen, scale=1.0 / B), _normal(B, d, gen)
    inv = torch.rsqrt(Z.double().square().mean(1) + EPS).float()
    return A, X, _glorot(d, d, gen), torch.rand(d, device=DEV, generator=gen) + 0.5, dY, Z, inv


def _prepare_block(case, seed):
    B, d = case["rows"], case["d"]
    (rowptr, colidx, val), X, W, gam, dY, Zb, inv = _inputs_block(case, seed)
    ctx = sg.Context(0)
    ctx.reserve(B, colidx.numel(), B, d, 2 * colidx.numel() + 16 * B + 65536)
    m = {k: _mat(B, d, torch.float32) for k in ("T", "Z", "Y", "dZ", "dT", "dX")}
    return dict(run=_run_block, case=case, ctx=ctx, A=_csr(ctx, B, rowptr, colidx, val), X=X, W=W, gam=gam, dY=dY, Zb=Zb, inv=inv,
                ir=torch.empty(B, device=DEV), dW=torch.empty_like(W), dg=torch.empty_like(gam), drop_seed=seed & M32, **m)


def _run_block(s):
    # The backward half works from a stored Z of its own: an entry of Z within rounding of zero would else flip its ReLU.
    c, ctx, A = s["case"], s["ctx"], s["A"]
    f = sg.SGNN_BF16_MFMA if c["bf16"] else 0
    sg.sgnn_spmm(ctx, A, s["X"], s["T"])
    sg.sgnn_gemm_tail_fwd(ctx, s["T"], s["W"], s["gam"], EPS, s["X"], c["drop"], s["drop_seed"], 1, 5, f, s["Z"], s["Y"], s["ir"])
    sg.sgnn_tail_bwd(ctx, s["Zb"], s["inv"], s["gam"], c["drop"], s["drop_seed"], 1, 5, s["dY"], s["dZ"], s["dg"], None)
    sg.sgnn_gemm(ctx, True, False, s["T"], s["dZ"], None, f, s["dW"])
    sg.sgnn_gemm(ctx, False, True, s["dZ"], s["W"], None, f, s["dT"])
    sg.sgnn_spmm(ctx, A, s["dT"], s["dX"], add=s["dY"])
    return dict(T=s["T"], Z=s["Z"], Y=s["Y"], ir=s["ir"], dZ=s["dZ"], dg=s["dg"], dW=s["dW"], dT=s["dT"], dX=s["dX"])


def _inputs_eval(case, seed):
    N, gen, dims = case["N"], _gen(seed, 5), _dims(case)
    rowptr, colidx = _graph(N, case["edges"], gen)
    X = torch.randn((N, dims[0]), device=DEV, generator=gen)
    return rowptr, colidx, X, [(_glorot(a, b, gen), _bias(b, gen)) for a, b in zip(dims, dims[1:])]


def _prepare_eval(case, seed):
    N = case["N"]
    rowptr, colidx, X, weights = _inputs_eval(case, seed)
    ctx = sg.Context(0)
    ctx.reserve(N, colidx.numel(), N, max(_dims(case)), colidx.numel())
    A = sg.sgnn_graph_normalized_csr(ctx, N, rowptr, colidx)
    bufs = [(torch.empty((N, W.shape[1]), device=DEV), torch.empty((N, W.shape[0]), device=DEV)) for W, _ in weights]
    return dict(run=_run_eval, ctx=ctx, A=A, X=X, weights=weights, bufs=bufs, bf16=case["bf16"])


def _run_eval(s):
    H = s["X"]
    for l, ((W, b), (Y, T)) in enumerate(zip(s["weights"], s["bufs"])):
        flags = (sg.SGNN_BF16_MFMA if s["bf16"] else 0) | (sg.SGNN_RELU if l + 1 < len(s["weights"]) else 0)
        if W.shape[1] < W.shape[0]:
            flags |= sg.SGNN_XFORM_FIRST
        sg.sgnn_gcn_fwd(s["ctx"], s["A"], H, W, b, flags, Y, T)
        H = Y
    return dict(hidden=s["bufs"][0][0], logits=H)


def _inputs_step(case, seed):
    N, gen, dims = case["N"], _gen(seed, 6), _dims(case)
    rowptr, colidx = _graph(N, case["edges"], gen)
    X = torch.randn((N, dims[0]), device=DEV, generator=gen)
    labels = torch.randint(0, dims[-1], (N,), device=DEV, dtype=torch.int32, generator=gen)
    return rowptr, colidx, X, labels, [(_glorot(a, b, gen), _bias(b, gen)) for a, b in zip(dims, dims[1:])]


def _prepare_step(case, seed):
    rowptr, colidx, X, labels, weights = _inputs_step(case, seed)
    st = sg.GcnStep(case["N"], rowptr, colidx, X, labels, weights, case["rows"], seed=seed, bf16=case["bf16"], bf16_activations=case["bf16"],
                    fuse_loss=True, keep_logits=case["logits"])
    return dict(run=_run_step, st=st, first=seed & 255, steps=case["steps"], logits=case["logits"] or not st.fuse_loss)


def _run_step(s):
    st, t = s["st"], s["first"]
    if s["steps"] == 1:
        st.step(t)
    else:
        st.run(range(t, t + s["steps"]))
    out = dict(loss=st.loss, dW=list(st.dW), db=list(st.db))
    if s["logits"]:
        out["logits"] = st.H[-1]
    return out


# ---------------------------------------------------------------------------------------------- work and tolerance

def _sampled(N, E, B):
    """Expected edges of the sampled rows, and entries of the induced matrix."""
    return E * B / N, B + (E - N) * (B / N) * ((B - 1) / max(N - 1, 1))


def _layer_work(rows, nnz, d_in, d_out, e, first, xform):
    csr, w = 8.0 * nnz + 4.0 * rows, 4.0 * d_in * d_out
    d_sp = d_out if xform else d_in
    fwd = csr + rows * e * (d_in + (0 if xform else d_in) + d_out) + w
    bwd = csr + rows * e * (d_in + d_out + (0 if first else 2 * d_in)) + 2 * w
    flops = 2.0 * nnz * d_sp + 2.0 * rows * d_in * d_out                                  # forward
    flops += 2.0 * rows * d_in * d_out * (1 if first else 2)                              # dW, and dT or dH
    flops += 0 if first and not xform else 2.0 * nnz * d_sp
    return fwd + bwd, flops


def _minibatch_bytes(N, E, B, i64):
    scanned, nnz = _sampled(N, E, B)
    return 4.0 * scanned + (16.0 if i64 else 8.0) * B + 16.0 * B + 3.0 * N / 16 + 8.0 * nnz


def work(case):
    k = case["kind"]
    e = 2 if case.get("bf16") else 4
    if k == "minibatch":
        N, E, B = case["N"], 2 * case["edges"] + case["N"], case["rows"]
        extra = 16.0 * _sampled(N, E, B)[1] / case["shard"] ** 2 if case["shard"] > 1 else 0.0
        return {"bytes": _minibatch_bytes(N, E, B, case["i64"]) + 8.0 * B * case["feat"] + extra, "flops": 0.0}
    if k == "eval":
        N, nnz, dims = case["N"], 2 * case["edges"] + case["N"], _dims(case)
        byt, flops = 0.0, 0.0
        for a, b in zip(dims, dims[1:]):
            byt += 8.0 * nnz + 4.0 * N * (a + b + (0 if b < a else a))
            flops += 2.0 * nnz * min(a, b) + 2.0 * N * a * b
        return {"bytes": byt, "flops": flops}
    if k == "block":
        B, nnz, d = case["rows"], case["rows"] * case["deg"], case["d"]
        # X, T, Z, Y; then Z, dY, dZ, T, dT, dX, dY once more
        return {"bytes": 16.0 * nnz + 4.0 * B * d * 11 + 12.0 * d * d, "flops": 4.0 * nnz * d + 6.0 * B * d * d}
    if k == "layer":
        byt, flops = _layer_work(case["rows"], case["rows"] * case["deg"], case["d_in"], case["d_out"], e, case["first"], case["xform"])
        return {"bytes": byt, "flops": flops}
    if k == "head":
        B, C = case["rows"], case["d_out"]
        byt, flops = _layer_work(B, B * case["deg"], case["d_in"], C, e, False, C < case["d_in"])
        keep = 4.0 * B * C if case["logits"] or not case["fused"] else 0.0
        return {"bytes": byt + keep + 4.0 * B, "flops": flops}
    N, E, B, dims = case["N"], 2 * case["edges"] + case["N"], case["rows"], _dims(case)
    byt, flops = _minibatch_bytes(N, E, B, True), 0.0
    for l, (a, b) in enumerate(zip(dims, dims[1:])):
        x, y = _layer_work(B, _sampled(N, E, B)[1], a, b, e, l == 0, b < a)
        byt, flops = byt + x, flops + y
    return {"bytes": byt * case["steps"], "flops": flops * case["steps"]}


def tolerance(case):
    if case["kind"] == "minibatch":
        return {"rel": 1e-6}      # the weights: a reciprocal square root in fp32; everything else is whole numbers
    if case["kind"] == "step":
        # a unit within rounding of zero may switch on or off: seldom in fp32, in one of some hundred rows in bfloat16
        return {"rel": 1.5e-2 if case["bf16"] else 5e-5}
    return {"rel": 1e-2 if case["bf16"] else 4e-6}


# ---------------------------------------------------------------------------------------------- the same in 64 bits

def _philox(c0, c1, c2, c3, k0, k1):
    """Philox4x32-10 on int64 tensors that hold 32-bit words."""
    for _ in range(10):
        p0, p1 = c0 * 0xD2511F53, c2 * 0xCD9E8D57
        c0, c1, c2, c3 = ((p1 >> 32) & M32) ^ c1 ^ k0, p1 & M32, ((p0 >> 32) & M32) ^ c3 ^ k1, p0 & M32
        k0, k1 = (k0 + 0x9E3779B9) & M32, (k1 + 0xBB67AE85) & M32
    return c0, c1, c2, c3


def _sample64(N, B, seed, step):
    j = torch.arange((N + 1) // 2, device=DEV)
    zero = torch.zeros_like(j)
    w = _philox(j, zero, zero + (step & M32), zero + (step >> 32), seed & M32, (seed >> 32) & M32)
    key = torch.stack([((w[1] - (1 << 31)) << 32) | w[0], ((w[3] - (1 << 31)) << 32) | w[2]], 1).reshape(-1)[:N]
    return torch.sort(torch.sort(key, stable=True)[1][:B])[0]


def _induce64(N, rowptr, colidx, S, rows=None, cols=None):
    """(row, col, val) of the normalised, rescaled matrix induced by S, in row order; rows / cols: vertex ranges that are kept."""
    B = S.numel()
    pos = torch.full((N,), -1, dtype=torch.int64, device=DEV)
    pos[S] = torch.arange(B, device=DEV)
    deg = rowptr[1:] - rowptr[:-1]
    n = deg[S]
    row = torch.repeat_interleave(torch.arange(B, device=DEV), n)
    flat = torch.arange(row.numel(), device=DEV) - torch.repeat_interleave(torch.cumsum(n, 0) - n, n) + torch.repeat_interleave(rowptr[:-1][S], n)
    u = colidx[flat].long()
    keep = pos[u] >= 0
    if rows is not None:
        v = S[row]
        keep &= (v >= rows[0]) & (v < rows[1]) & (u >= cols[0]) & (u < cols[1])
    row, u = row[keep], u[keep]
    val = torch.rsqrt(deg[S[row]].double() * deg[u].double())
    return row, pos[u], torch.where(S[row] == u, val, val * ((N - 1) / max(B - 1, 1)))


def _spmm64(A, X, rows):
    row, col, val = A
    out = torch.zeros((rows, X.shape[1]), dtype=torch.float64, device=DEV)
    step = max(1, (1 << 27) // X.shape[1])
    for a in range(0, row.numel(), step):
        b = a + step
        out.index_add_(0, row[a:b], X[col[a:b]].double() * val[a:b, None])
    return out


def _coo(A):
    rowptr, colidx, val = A
    n = (rowptr[1:] - rowptr[:-1]).long()
    return torch.repeat_interleave(torch.arange(n.numel(), device=DEV), n), colidx.long(), val.double()


def exact(case, seed):
    return globals()["_exact_" + case["kind"]](case, seed)


def _exact_minibatch(case, seed):
    rowptr, colidx, labels, X = _inputs_minibatch(case, seed)
    N, B = case["N"], case["rows"]
    S = _sample64(N, B, seed, seed & 255)
    r0, r1, c0, c1 = _tile(case)
    row, col, v = _induce64(N, rowptr, colidx, S, (r0, r1), (c0, c1))
    cap = _capacity(N, colidx.numel(), B)

    def padded(x):
        out = torch.zeros(max(cap, 1), dtype=torch.float64, device=DEV)
        out[:x.numel()] = x
        return out
    out = dict(S=None, bitmap=None, rank=None, rowptr=None, colidx=None, val=padded(v), nnz=None, y=None)
    if case["shard"] > 1:
        out.update(t_rowptr=None, t_colidx=None, t_val=padded(v[torch.sort(col * B + row)[1]]))
    if X is not None:
        out["X_S"] = X[S].double()
    return out


def _exact_layer(case, seed):
    A, S, H, W, b, dY = _inputs_layer(case, seed)
    A, B, W, dY = _coo(A), case["rows"], W.double(), dY.double()
    X = (H if S is None else H[S.long()]).double()
    if case["xform"]:
        Y, saved = _spmm64(A, X @ W, B), X
        dP = _spmm64(A, dY, B)                 # the matrix is symmetric
    else:
        saved = _spmm64(A, X, B)
        Y, dP = saved @ W, dY
    out = dict(Y=(Y + b.double()).relu_(), dW=saved.T @ dP, db=dY.sum(0))
    if not case["xform"]:
        out["T"] = saved
    if not case["first"]:
        dH = dP @ W.T
        out["dH"] = (dH if case["xform"] else _spmm64(A, dH, B)) * (H > 0)
    return out


def _exact_head(case, seed):
    A, H, W, b, y = _inputs_head(case, seed)
    A, B, W, X = _coo(A), case["rows"], W.double(), H.double()
    xform = case["d_out"] < case["d_in"]
    T = None if xform else _spmm64(A, X, B)
    logits = (_spmm64(A, X @ W, B) if xform else T @ W) + b.double()
    y = y.long()[:, None]
    loss = (torch.logsumexp(logits, 1, keepdim=True) - logits.gather(1, y)).mean()
    dO = torch.softmax(logits, 1).scatter_add_(1, y, torch.full(y.shape, -1.0, dtype=torch.float64, device=DEV)) / B
    dP = _spmm64(A, dO, B) if xform else dO
    dH = dP @ W.T
    out = dict(loss=loss.reshape(1), dO=dO, db=dO.sum(0), dW=(X if xform else T).T @ dP,
               dH=(dH if xform else _spmm64(A, dH, B)) * (H > 0))
    if case["logits"] or not (xform and case["fused"]):
        out["O"] = logits
    return out


def _exact_block(case, seed):
    A, X, W, gam, dY, Zb, inv = _inputs_block(case, seed)
    B, d, q, drop_seed = case["rows"], case["d"], case["drop"], seed & M32
    A, Xd, W, gam, dYd = _coo(A), X.double(), W.double(), gam.double(), dY.double()
    keep = torch.ones((B, d), dtype=torch.float64, device=DEV)
    if q > 0:
        blk = torch.arange((B * d + 3) // 4, device=DEV)
        zero = torch.zeros_like(blk)
        w = torch.stack(_philox(blk & M32, blk >> 32, zero + 5, zero + (1 << 31) + 1, drop_seed, 0), 1).reshape(-1)[:B * d].reshape(B, d)
        q32 = float(torch.tensor(q, dtype=torch.float32))
        keep = (w >= int(q32 * 2 ** 32)).double() / (1.0 - q32)
    T = _spmm64(A, Xd, B)
    Z = T @ W
    ir = torch.rsqrt(Z.square().mean(1) + EPS)
    Y = (gam * Z * ir[:, None]).relu_() * keep + Xd
    Zd, ivd = Zb.double(), inv.double()[:, None]
    nrm = Zd * ivd
    g = dYd * keep * (gam * nrm > 0)
    dg = (g * nrm).sum(0)
    t = g * gam
    dZ = ivd * (t - nrm * (t * nrm).mean(1, keepdim=True))
    dT = dZ @ W.T
    return dict(T=T, Z=Z, Y=Y, ir=ir, dZ=dZ, dg=dg, dW=T.T @ dZ, dT=dT, dX=_spmm64(A, dT, B) + dYd)


def _exact_eval(case, seed):
    rowptr, colidx, X, weights = _inputs_eval(case, seed)
    N = case["N"]
    deg = rowptr[1:] - rowptr[:-1]
    row, col = torch.repeat_interleave(torch.arange(N, device=DEV), deg), colidx.long()
    A = row, col, torch.rsqrt(deg[row].double() * deg[col].double())
    H, hidden = X.double(), []
    for l, (W, b) in enumerate(weights):
        W = W.double()
        H = (_spmm64(A, H @ W, N) if W.shape[1] < W.shape[0] else _spmm64(A, H, N) @ W) + b.double()
        H = H.relu_() if l + 1 < len(weights) else H
        hidden.append(H)
    return dict(hidden=hidden[0], logits=H)


def _exact_step(case, seed):
    rowptr, colidx, X, labels, weights = _inputs_step(case, seed)
    N, B, dims = case["N"], case["rows"], _dims(case)
    S = _sample64(N, B, seed, (seed & 255) + case["steps"] - 1)
    A = _induce64(N, rowptr, colidx, S)
    y = labels[S].long()[:, None]
    H, saved, L = [X[S].double()], [], len(weights)
    for l, (W, b) in enumerate(weights):
        W, xform = W.double(), dims[l + 1] < dims[l]
        saved.append(H[l] if xform else _spmm64(A, H[l], B))
        Z = (_spmm64(A, H[l] @ W, B) if xform else saved[l] @ W) + b.double()
        H.append(Z.relu_() if l + 1 < L else Z)
    loss = (torch.logsumexp(H[L], 1, keepdim=True) - H[L].gather(1, y)).mean()
    dZ = torch.softmax(H[L], 1).scatter_add_(1, y, torch.full(y.shape, -1.0, dtype=torch.float64, device=DEV)) / B
    dW, db = [None] * L, [None] * L
    for l in range(L - 1, -1, -1):
        W, xform = weights[l][0].double(), dims[l + 1] < dims[l]
        db[l] = dZ.sum(0)
        dP = _spmm64(A, dZ, B) if xform else dZ
        dW[l] = saved[l].T @ dP
        if l:
            dH = dP @ W.T
            dZ = (dH if xform else _spmm64(A, dH, B)) * (H[l] > 0)
    out = dict(loss=loss.reshape(1), dW=dW, db=db)
    if case["logits"] or dims[-1] >= dims[-2]:
        out["logits"] = H[L]
    return out
