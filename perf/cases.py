"""Performance cases of the shard library: what one GPU of a replica does in a training step, through the entry points of
paper_2504_06095_amd, from the smallest shard to the largest layer.

A case is a dict of plain values; its "kind" names the path:
  mlp       MLP shard, forward + backward, `micro` micro-batches whose gradients accumulate
  attn      attention shard of a rank's heads: projections and core, forward + backward
  core      the attention core alone, forward (+ backward)
  layer     a whole layer shard, forward + backward, the weight gradients stored into the full-TP layout by the gradient GEMMs
  reshard   one layer's tensors, all ranks on this GPU, between two contiguous TP layouts
  mapped    the same between the compute and sync layouts of the shard-mapping algorithm, through prepared plans
"""
import math

import torch

import paper_2504_06095_amd as N

K = N.binding
BF, F32 = torch.bfloat16, torch.float32
ACT, WEIGHT, GRAD = 1.0, 0.02, 1.0e-3  # standard deviations of activations and upstream gradients, weights, weight gradients


def listed():
    return [
        # a small model's FFN shard at TP 8 -> 7: launches and latency
        dict(name="mlp_small", kind="mlp", tokens=512, hidden=1024, width=586, gelu="erf", micro=1, pad=64),
        # GPT-3-175B-shape FFN shard at TP 8 -> 7
        dict(name="mlp_gpt3", kind="mlp", tokens=2048, hidden=12288, width=7022, gelu="erf", micro=1, pad=64),
        # 405B-shape FFN at TP 72 -> 71: many tokens, a narrow ragged shard
        dict(name="mlp_405b", kind="mlp", tokens=8192, hidden=16384, width=750, gelu="erf", micro=1, pad=64),
        # hidden 6144 at TP 8 -> 7, two micro-batches before the sync, tanh GeLU, rows padded only as far as required
        dict(name="mlp_accumulate", kind="mlp", tokens=4096, hidden=6144, width=3511, gelu="tanh", micro=2, pad=8),
        # grouped-query attention shard at TP 32 -> 30, first rank (3 heads over one KV head)
        dict(name="attn_gqa", kind="attn", n_seq=1, seq=4096, hidden=8192, n_q=64, n_kv=8, dim=128, tp=30, rank=0, causal=True),
        # a small model's attention shard (16 heads of 64) at TP 8 -> 7, four sequences
        dict(name="attn_small", kind="attn", n_seq=4, seq=512, hidden=1024, n_q=16, n_kv=16, dim=64, tp=7, rank=0, causal=True),
        # attention core of the GPT-3-175B-shape shard, one 2048-token sequence
        dict(name="core_2k", kind="core", n_seq=1, seq=2048, heads=14, kv=14, dim=128, causal=True, back=True),
        # the same heads over a long sequence, unmasked as the paper writes it
        dict(name="core_8k", kind="core", n_seq=1, seq=8192, heads=14, kv=14, dim=128, causal=False, back=True),
        # GPT-3-175B-shape layer shard at TP 8 -> 7, gradients into the TP-8 layout
        dict(name="layer_gpt3", kind="layer", seq=2048, hidden=12288, ffn=49152, n_q=96, n_kv=96, dim=128, tp=7, full=8),
        # 405B-shape layer's fp32 weight gradients, TP 71 -> 72
        dict(name="reshard_405b", kind="reshard", hidden=16384, ffn=53248, n_q=128, n_kv=8, dim=128, src=71, dst=72, elem=4),
        # GPT-3-175B-shape layer's bf16 weights when a replica drops from TP 8 to TP 7
        dict(name="reshard_weights", kind="reshard", hidden=12288, ffn=49152, n_q=96, n_kv=96, dim=128, src=8, dst=7, elem=2),
        # hidden 12288 layer's gradients of a healthy TP-32 replica, compute layout -> the TP-30 sync layout
        dict(name="mapped_sync", kind="mapped", hidden=12288, ffn=49152, heads=96, dim=128, full=32, tp=30, back=False),
    ]


# What a drawn case may cost at most: the work of the listed layer shard, the traffic of the listed 405B-shape reshard.
MAX_FLOPS, MAX_BYTES = 2.0e12, 1.2e10


def _log(rng, lo, hi):
    return math.exp(rng.uniform(math.log(lo), math.log(hi)))


def _shard(dim, tp):
    return N.ntp_shard_plan(dim, tp, 0)[1]


def _draw(rng, kind):
    if kind == "mlp":
        hidden = 8 * round(_log(rng, 512, 16384) / 8)
        return dict(kind=kind, tokens=round(_log(rng, 128, 16384)), hidden=hidden, width=_shard(4 * hidden, rng.choice((3, 4, 6, 7, 11, 30, 71))),
                    gelu=rng.choice(("erf", "erf", "tanh")), micro=rng.choice((1, 1, 2)), pad=rng.choice((8, 64)))
    if kind == "attn":
        dim = rng.choice((64, 128, 128))
        kv = rng.choice((2, 4, 8, 16))
        n_q = kv * rng.choice((1, 2, 4, 8))
        tp = rng.randint(2, max(2, n_q // 2))
        return dict(kind=kind, n_seq=rng.choice((1, 1, 2, 4)), seq=round(_log(rng, 128, 8192)), hidden=64 * round(_log(rng, 512, 12288) / 64),
                    n_q=n_q, n_kv=kv, dim=dim, tp=tp, rank=rng.randrange(tp), causal=rng.random() < 0.75)
    if kind == "core":
        kv = rng.choice((1, 2, 3, 4, 7, 14))
        return dict(kind=kind, n_seq=rng.choice((1, 1, 2, 4)), seq=round(_log(rng, 256, 16384)), heads=kv * rng.choice((1, 1, 2, 4)), kv=kv,
                    dim=rng.choice((64, 128, 128)), causal=rng.random() < 0.7, back=rng.random() < 0.75)
    if kind == "layer":
        dim = rng.choice((64, 128, 128))
        heads = rng.randint(8, 96)
        full = rng.choice((4, 8))
        return dict(kind=kind, seq=round(_log(rng, 256, 8192)), hidden=heads * dim, ffn=4 * heads * dim, n_q=heads, n_kv=heads, dim=dim,
                    tp=rng.randint(full // 2, full - 1), full=full)
    dim = 128
    heads = rng.randint(8, 128)
    hidden = heads * dim
    full = rng.randint(4, min(72, heads))
    tp = rng.randint(max(2, full * 3 // 4), full - 1)
    if kind == "reshard":
        a, b = rng.choice(((tp, full), (full, tp)))
        return dict(kind=kind, hidden=hidden, ffn=4 * hidden, n_q=heads, n_kv=rng.choice([k for k in (1, 2, 4, 8, heads) if heads % k == 0]),
                    dim=dim, src=a, dst=b, elem=rng.choice((2, 4)))
    return dict(kind=kind, hidden=hidden, ffn=4 * hidden, heads=heads, dim=dim, full=full, tp=tp, back=rng.random() < 0.5)


def draw(rng):
    kind = rng.choice(("mlp", "mlp", "attn", "core", "layer", "reshard", "mapped"))
    while True:
        case = _draw(rng, kind)
        w = work(case)
        if w["flops"] <= MAX_FLOPS and w["bytes"] <= MAX_BYTES:
            return case


# ---- buffers -------------------------------------------------------------------------------------
class _Make:
    """Seeded normal device tensors, bf16 unless said otherwise."""

    def __init__(self, seed):
        self.gen = torch.Generator("cuda")
        self.gen.manual_seed(seed)

    def __call__(self, rows, cols, std, dtype=BF):
        return torch.empty(rows, cols, dtype=dtype, device="cuda").normal_(0.0, std, generator=self.gen)

    def flat(self, n, dtype, std):
        t = torch.empty(n, dtype=dtype, device="cuda")
        for i in range(0, n, 1 << 28):
            t[i : i + (1 << 28)].normal_(0.0, std, generator=self.gen)
        return t


def _empty(rows, cols, dtype=BF):
    return torch.empty(rows, cols, dtype=dtype, device="cuda")


def _padded(rows, width, pad):
    """[rows x width] view whose rows are `pad`-aligned; zeroed so that nothing unwritten is ever read."""
    return torch.zeros(rows, -(-width // pad) * pad, dtype=BF, device="cuda")[:, :width]


def _handle(*calls):
    """A handle with as much workspace as any of the (call, shape) pairs can use."""
    h = N.ntp_create()
    n = max(N.ntp_workspace_bytes(c, s, handle=h) for c, s in calls)
    if n:
        N.ntp_set_workspace(torch.empty(n, dtype=torch.uint8, device="cuda"), handle=h)
    return h


class _Mlp:
    def __init__(self, make, tokens, hidden, width, gelu, pad, micro=1, grads=True):
        self.n_r, self.mode = width, K.NTP_GELU_TANH if gelu == "tanh" else K.NTP_GELU_ERF
        self.X = [make(tokens, hidden, ACT) for _ in range(micro)]
        self.dZ = [make(tokens, hidden, ACT) for _ in range(micro)]
        self.At, self.B = make(width, hidden, WEIGHT), make(width, hidden, WEIGHT)
        self.P, self.Y, self.dP = (_padded(tokens, width, pad) for _ in range(3))
        self.Z = [_empty(tokens, hidden) for _ in range(micro)]
        self.dX = [_empty(tokens, hidden) for _ in range(micro)]
        if grads:
            self.dA, self.dB = _empty(width, hidden, F32), _empty(width, hidden, F32)
        self.call = (K.NTP_CALL_MLP_SHARD, K.MlpShape(tokens, hidden, width, self.mode))

    def fwd(self, h, i):
        N.ntp_mlp_shard_fwd(self.X[i], self.At, self.B, self.P, self.Y, self.Z[i], self.n_r, self.mode, handle=h)

    def bwd(self, h, i):
        N.ntp_mlp_shard_bwd(self.dZ[i], self.X[i], self.At, self.B, self.P, self.Y, self.dP, self.dX[i], self.dA, self.dB, self.n_r,
                            self.mode, accumulate=i > 0, handle=h)

    def bwd_resharded(self, h, seg_a, seg_b):
        N.ntp_mlp_shard_bwd_resharded(self.dZ[0], self.X[0], self.At, self.B, self.P, self.Y, self.dP, self.dX[0], seg_a, seg_b, self.n_r,
                                      self.mode, handle=h)


class _Core:
    def __init__(self, n_seq, seq, plan, group, causal):
        self.shape = N.attn_core_shape(n_seq, seq, plan, group, causal)
        m = n_seq * seq
        self.C, self.LSE, self.Delta = _empty(m, plan["w_o"]), _empty(plan["q_cnt"], m, F32), _empty(plan["q_cnt"], m, F32)
        self.dQKV = _empty(m, plan["w_qkv"])
        self.call = (K.NTP_CALL_ATTN_CORE_SHARD, self.shape)

    def fwd(self, h, QKV):
        N.ntp_attn_core_shard_fwd(self.shape, QKV, self.C, self.LSE, handle=h)

    def bwd(self, h, QKV, dC):
        N.ntp_attn_core_shard_bwd(self.shape, QKV, self.C, dC, self.LSE, self.Delta, self.dQKV, handle=h)


class _Attn:
    def __init__(self, make, n_seq, seq, hidden, plan, group, causal, grads=True):
        self.core = _Core(n_seq, seq, plan, group, causal)
        m, wq, wo = n_seq * seq, plan["w_qkv"], plan["w_o"]
        self.dims = (m, hidden, wq, wo)
        self.X, self.dZ = make(m, hidden, ACT), make(m, hidden, ACT)
        self.Wqkv, self.Wo = make(wq, hidden, WEIGHT), make(wo, hidden, WEIGHT)
        self.QKV, self.Z, self.dC, self.dX = _empty(m, wq), _empty(m, hidden), _empty(m, wo), _empty(m, hidden)
        if grads:
            self.dWqkv, self.dWo = _empty(wq, hidden, F32), _empty(wo, hidden, F32)
        self.calls = (self.core.call, (K.NTP_CALL_ATTN_PROJ_SHARD, K.AttnShape(*self.dims)))

    def fwd(self, h):
        N.ntp_attn_proj_shard_fwd(*self.dims, X=self.X, Wqkv=self.Wqkv, QKV=self.QKV, handle=h)
        self.core.fwd(h, self.QKV)
        N.ntp_attn_proj_shard_fwd(*self.dims, C_=self.core.C, Wo=self.Wo, Zpart=self.Z, handle=h)

    def bwd(self, h):
        N.ntp_attn_proj_shard_bwd(*self.dims, dZ=self.dZ, C_=self.core.C, Wo=self.Wo, dC=self.dC, dWo=self.dWo, handle=h)
        self.core.bwd(h, self.QKV, self.dC)
        N.ntp_attn_proj_shard_bwd(*self.dims, dQKV=self.core.dQKV, X=self.X, Wqkv=self.Wqkv, dXpart=self.dX, dWqkv=self.dWqkv, handle=h)

    def bwd_resharded(self, h, seg_qkv, seg_o):
        N.ntp_attn_proj_shard_bwd_resharded(*self.dims, dZ=self.dZ, C_=self.core.C, Wo=self.Wo, dC=self.dC, dWo_segs=seg_o, handle=h)
        self.core.bwd(h, self.QKV, self.dC)
        N.ntp_attn_proj_shard_bwd_resharded(*self.dims, dQKV=self.core.dQKV, X=self.X, Wqkv=self.Wqkv, dXpart=self.dX, dWqkv_segs=seg_qkv,
                                            handle=h)


def _tensors(case, elem):
    """The four weights (or gradients) of a layer: fc1 and QKV as the paper writes them [hidden x width], cut by columns; fc2 and the output
    projection cut by rows.  (spec, width of a rank's shard along the cut axis as a function of (tp, rank))."""
    hd, f, q, kv, d = (case[k] for k in ("hidden", "ffn", "n_q", "n_kv", "dim"))
    even = lambda dim, unit: lambda tp, r: N.ntp_shard_plan(dim // unit, tp, r)[1] * unit  # noqa: E731
    return [(N.tensor_spec(hd, f, 1, 1, elem), even(f, 1)),
            (N.tensor_spec(f, hd, 0, 1, elem), even(f, 1)),
            (N.tensor_spec(hd, (q + 2 * kv) * d, 1, d, elem, K.NTP_KIND_QKV_GQA, q, kv), lambda tp, r: N.ntp_attn_shard_plan(q, kv, d, tp, r)["w_qkv"]),
            (N.tensor_spec(q * d, hd, 0, d, elem), even(q * d, d))]


def _views(shapes, elem, fill):
    """One buffer for all shards of a tensor (a gradient bucket), every shard dense and 256-byte aligned in it; the shards' views."""
    at, total = [], 0
    for r, c in shapes:
        at.append(total)
        total += -(-r * c * elem // 256) * 256 // elem
    buf = fill(max(total, 1))
    return buf, [buf[o : o + r * c].view(r, c) if r * c else None for o, (r, c) in zip(at, shapes)]


def _cut(spec, widths):
    return [(spec.rows, w) if spec.partition_dim else (w, spec.cols) for w in widths]


# ---- the measured interface ------------------------------------------------------------------------
def prepare(case, seed):
    make, kind = _Make(seed), case["kind"]
    s = dict(kind=kind)
    if kind == "mlp":
        s["mlp"] = _Mlp(make, case["tokens"], case["hidden"], case["width"], case["gelu"], case["pad"], case["micro"])
        s["h"] = _handle(s["mlp"].call)
    elif kind == "attn":
        plan = N.ntp_attn_shard_plan(case["n_q"], case["n_kv"], case["dim"], case["tp"], case["rank"])
        s["attn"] = _Attn(make, case["n_seq"], case["seq"], case["hidden"], plan, case["n_q"] // case["n_kv"], case["causal"])
        s["h"] = _handle(*s["attn"].calls)
    elif kind == "core":
        plan = N.ntp_attn_shard_plan(case["heads"], case["kv"], case["dim"], 1, 0)
        s["core"] = _Core(case["n_seq"], case["seq"], plan, case["heads"] // case["kv"], case["causal"])
        m = case["n_seq"] * case["seq"]
        s["QKV"] = make(m, plan["w_qkv"], ACT)
        s["dC"] = make(m, plan["w_o"], ACT) if case["back"] else None
        s["h"] = _handle(s["core"].call)
    elif kind == "layer":
        tp, full, hd = case["tp"], case["full"], case["hidden"]
        plan = N.ntp_attn_shard_plan(case["n_q"], case["n_kv"], case["dim"], tp, 0)
        s["attn"] = _Attn(make, 1, case["seq"], hd, plan, case["n_q"] // case["n_kv"], True, grads=False)
        s["mlp"] = _Mlp(make, case["seq"], hd, _shard(case["ffn"], tp), "erf", 64, grads=False)
        s["h"] = _handle(*s["attn"].calls, s["mlp"].call)
        s["shards"], s["segs"] = [], []
        q, kv, d, f = case["n_q"], case["n_kv"], case["dim"], case["ffn"]
        for spec in (N.tensor_spec((q + 2 * kv) * d, hd, 0, d, 4, K.NTP_KIND_QKV_GQA, q, kv), N.tensor_spec(q * d, hd, 0, d, 4),
                     N.tensor_spec(f, hd, 0, 1, 4), N.tensor_spec(f, hd, 0, 1, 4)):
            mine = {seg[1] for seg in N.ntp_reshard_segments(spec, tp, full) if seg[0] == 0}
            dst = [None] * full
            for r in mine:
                rows = N.ntp_attn_shard_plan(q, kv, d, full, r)["w_qkv"] if spec.kind else N.ntp_shard_plan(spec.rows // spec.unit, full, r)[1] * spec.unit
                dst[r] = torch.zeros(rows, hd, dtype=F32, device="cuda")  # rows that other ranks send stay zero
            s["shards"].append([t for t in dst if t is not None])
            s["segs"].append(N.ntp_reshard_row_segments(spec, tp, 0, full, dst))
    elif kind == "reshard":
        dtype, std = (F32, GRAD) if case["elem"] == 4 else (BF, WEIGHT)
        s.update(src=case["src"], dst=case["dst"], jobs=[], out=[], h=N.ntp_create())
        for spec, width in _tensors(case, case["elem"]):
            full = make.flat(spec.rows * spec.cols, dtype, std).view(spec.rows, spec.cols)
            _, srcs = _views(_cut(spec, [width(case["src"], r) for r in range(case["src"])]), case["elem"],
                             lambda n: torch.zeros(n, dtype=dtype, device="cuda"))
            _scatter(spec, case["src"], full, srcs)
            del full
            out, dsts = _views(_cut(spec, [width(case["dst"], r) for r in range(case["dst"])]), case["elem"],
                               lambda n: torch.zeros(n, dtype=dtype, device="cuda"))
            s["jobs"].append((spec, srcs, dsts))
            s["out"].append(out)
    else:
        full, tp = case["full"], case["tp"]
        s.update(jobs=[], out=[], h=N.ntp_create())
        hd, f, qd = case["hidden"], case["ffn"], case["heads"] * case["dim"]
        for rows, cols, pd, unit in ((hd, f, 1, 1), (f, hd, 0, 1), (qd, hd, 0, case["dim"])):
            k = (cols if pd else rows) // unit
            comp, sync = N.ntp_comp_sync_plan(k, full, tp)
            spec = N.tensor_spec(rows, cols, pd, unit, 4)
            (a, na), (b, nb) = ((sync, tp), (comp, full)) if case["back"] else ((comp, full), (sync, tp))
            counts = lambda ranks, n: torch.bincount(torch.tensor(ranks), minlength=n).mul(unit).tolist()  # noqa: E731
            _, srcs = _views(_cut(spec, counts(a, na)), 4, lambda n: make.flat(n, F32, GRAD))
            out, dsts = _views(_cut(spec, counts(b, nb)), 4, lambda n: torch.zeros(n, dtype=F32, device="cuda"))
            plan = N.ntp_reshard_plan_create(spec, na, a, nb, b)
            plan.ntp_reshard_plan_prepare()
            s["jobs"].append((plan, srcs, dsts))
            s["out"].append(out)
    return s


def _scatter(spec, tp, full, shards):
    """Cut a logical tensor into its TP = tp shards (a KV head that several ranks hold goes to each of them)."""
    u, cols = spec.unit, spec.partition_dim == 1
    for r, t in enumerate(shards):
        if t is None:
            continue
        if spec.kind:
            p = N.ntp_attn_shard_plan(spec.n_q, spec.n_kv, u, tp, r)
            runs = [(p["q_off"], p["q_cnt"]), (spec.n_q + p["kv_off"], p["kv_cnt"]), (spec.n_q + spec.n_kv + p["kv_off"], p["kv_cnt"])]
        else:
            runs = [N.ntp_shard_plan((spec.cols if cols else spec.rows) // u, tp, r)]
        at = 0
        for off, n in runs:
            if cols:
                t[:, at : at + n * u] = full[:, off * u : (off + n) * u]
            else:
                t[at : at + n * u] = full[off * u : (off + n) * u]
            at += n * u


def run(state):
    kind, h = state["kind"], state["h"]
    if kind == "mlp":
        m = state["mlp"]
        for i in range(len(m.X)):
            m.fwd(h, i)
            m.bwd(h, i)
        return dict(P=m.P, Y=m.Y, dP=m.dP, Z=m.Z, dX=m.dX, dA=m.dA, dB=m.dB)
    if kind == "attn":
        a = state["attn"]
        a.fwd(h)
        a.bwd(h)
        return dict(QKV=a.QKV, C=a.core.C, LSE=a.core.LSE, Z=a.Z, dC=a.dC, dQKV=a.core.dQKV, dX=a.dX, dWqkv=a.dWqkv, dWo=a.dWo)
    if kind == "core":
        c = state["core"]
        c.fwd(h, state["QKV"])
        if state["dC"] is None:
            return dict(C=c.C, LSE=c.LSE)
        c.bwd(h, state["QKV"], state["dC"])
        return dict(C=c.C, LSE=c.LSE, dQKV=c.dQKV)
    if kind == "layer":
        a, m = state["attn"], state["mlp"]
        seg_qkv, seg_o, seg_a, seg_b = state["segs"]
        a.fwd(h)
        m.fwd(h, 0)
        m.bwd_resharded(h, seg_a, seg_b)
        a.bwd_resharded(h, seg_qkv, seg_o)
        return dict(Zattn=a.Z, Zmlp=m.Z, dXmlp=m.dX, dXattn=a.dX, C=a.core.C, dQKV=a.core.dQKV, grads=state["shards"])
    if kind == "reshard":
        for spec, srcs, dsts in state["jobs"]:
            N.ntp_reshard_grad(spec, state["src"], state["dst"], srcs, dsts, handle=h)
    else:
        for plan, srcs, dsts in state["jobs"]:
            plan.ntp_reshard_plan_run(srcs, dsts, handle=h)
    return state["out"]


def _mlp_work(tokens, hidden, width, micro):
    act, wide, weight = 2 * tokens * hidden, 2 * tokens * width, width * hidden
    # X, dZ in, Z, dX out; P, Y, dP out; A, B in (bf16) and dA, dB out (fp32)
    return 12.0 * tokens * hidden * width * micro, micro * (4 * act + 3 * wide) + 2 * 2 * weight + 2 * 4 * weight


def _core_work(n_seq, seq, heads, kv, dim, causal, back):
    m = n_seq * seq
    pairs = n_seq * (seq * (seq + 1) / 2 if causal else float(seq) * seq)
    qkv, c = 2.0 * m * (heads + 2 * kv) * dim, 2.0 * m * heads * dim
    # products over head_dim: 2 forward, 5 backward
    return 2.0 * pairs * dim * heads * (7 if back else 2), qkv + c + 4 * heads * m + (c + qkv if back else 0)


def _attn_work(m, hidden, wq, wo):
    weight = (wq + wo) * hidden
    return 6.0 * m * weight, 4 * 2.0 * m * hidden + 2.0 * m * (wq + wo) * 2 + (2 + 4) * weight


def work(case):
    kind = case["kind"]
    if kind == "mlp":
        flops, nbytes = _mlp_work(case["tokens"], case["hidden"], case["width"], case["micro"])
    elif kind in ("attn", "layer"):
        rank, causal, n_seq = case.get("rank", 0), case.get("causal", True), case.get("n_seq", 1)
        p = N.ntp_attn_shard_plan(case["n_q"], case["n_kv"], case["dim"], case["tp"], rank)
        flops, nbytes = _attn_work(n_seq * case["seq"], case["hidden"], p["w_qkv"], p["w_o"])
        flops += _core_work(n_seq, case["seq"], p["q_cnt"], p["kv_cnt"], case["dim"], causal, True)[0]
        nbytes += 4.0 * p["q_cnt"] * n_seq * case["seq"]
        if kind == "layer":
            f, b = _mlp_work(case["seq"], case["hidden"], _shard(case["ffn"], case["tp"]), 1)
            flops, nbytes = flops + f, nbytes + b
    elif kind == "core":
        flops, nbytes = _core_work(*(case[k] for k in ("n_seq", "seq", "heads", "kv", "dim", "causal", "back")))
    else:
        hd, f, d, q = case["hidden"], case["ffn"], case["dim"], case.get("n_q", case.get("heads"))
        flops, nbytes = 0.0, 2.0 * f * hd + q * d * hd
        if kind == "reshard":
            kv = case["n_kv"]
            wide = sum(N.ntp_attn_shard_plan(q, kv, d, case["dst"], r)["w_qkv"] for r in range(case["dst"]))
            nbytes += (wide + (q + 2 * kv) * d) / 2.0 * hd  # every unit read once, every copy written
        nbytes *= 2 * case.get("elem", 4)
    return dict(bytes=nbytes, flops=flops)


def tolerance(case):
    if case["kind"] in ("reshard", "mapped"):
        return "exact"
    # bf16 results of fp32 sums
    return dict(rel=1e-2)


# ---- the same in 64 bits, plain torch --------------------------------------------------------------
def _d(t):
    return t.double()


def _mlp64(m):
    dA, dB, Z, dX = 0.0, 0.0, [], []
    At, B = _d(m.At), _d(m.B)
    for X, dZ in zip(map(_d, m.X), map(_d, m.dZ)):
        P = (X @ At.T).requires_grad_()
        Y = torch.nn.functional.gelu(P, approximate="tanh" if m.mode == K.NTP_GELU_TANH else "none")
        (dP,) = torch.autograd.grad(Y, P, dZ @ B.T)
        P, Y = P.detach(), Y.detach()
        Z.append(Y @ B)
        dX.append(dP @ At)
        dA, dB = dA + dP.T @ X, dB + Y.T @ dZ
    return dict(P=P, Y=Y, dP=dP, Z=Z, dX=dX, dA=dA, dB=dB)


def _core64(n_seq, seq, q, kv, head_of, dim, causal, QKV, dC):
    """`head_of[j]`: the local KV head that local query head j reads."""
    m, scale = n_seq * seq, 1.0 / math.sqrt(dim)
    C, dQKV = QKV.new_zeros(m, q * dim), torch.zeros_like(QKV)
    LSE = QKV.new_zeros(q, m)
    future = torch.ones(seq, seq, dtype=torch.bool, device=QKV.device).triu_(1) if causal else None
    for i in range(n_seq):
        rows = slice(i * seq, (i + 1) * seq)
        for j in range(q):
            cq, ck, cv = (slice(b * dim, (b + 1) * dim) for b in (j, q + head_of[j], q + kv + head_of[j]))
            Q, Kh, V = QKV[rows, cq], QKV[rows, ck], QKV[rows, cv]
            S = Q @ Kh.T * scale
            if causal:
                S.masked_fill_(future, -math.inf)
            LSE[j, rows] = lse = torch.logsumexp(S, 1)
            P = S.sub_(lse[:, None]).exp_()
            C[rows, cq] = O = P @ V
            if dC is not None:
                dO = dC[rows, cq]
                dQKV[rows, cv] += P.T @ dO
                dS = P * (dO @ V.T - (dO * O).sum(1, keepdim=True)) * scale
                dQKV[rows, cq] = dS @ Kh
                dQKV[rows, ck] += dS.T @ Q
    return C, LSE, dQKV


def _attn64(case, a):
    p = N.ntp_attn_shard_plan(case["n_q"], case["n_kv"], case["dim"], case["tp"], case.get("rank", 0))
    group = case["n_q"] // case["n_kv"]
    head_of = [(p["q_off"] + j) // group - p["kv_off"] for j in range(p["q_cnt"])]
    X, dZ, Wqkv, Wo = map(_d, (a.X, a.dZ, a.Wqkv, a.Wo))
    QKV, dC = X @ Wqkv.T, dZ @ Wo.T
    C, LSE, dQKV = _core64(case.get("n_seq", 1), case["seq"], p["q_cnt"], p["kv_cnt"], head_of, case["dim"], case.get("causal", True), QKV, dC)
    return dict(QKV=QKV, C=C, LSE=LSE, Z=C @ Wo, dC=dC, dQKV=dQKV, dX=dQKV @ Wqkv, dWqkv=dQKV.T @ X, dWo=C.T @ dZ)


def _own(n, tp, r):
    lo = r * (n // tp) + min(r, n % tp)
    return lo, lo + n // tp + (r < n % tp)


def _full_shards(dW, blocks, unit, n, full):
    """The parts of the TP = full shards that lie in rank 0's rows: `blocks` blocks of n units a tensor, rank 0's first units of each in dW."""
    mine, out = dW.view(blocks, -1, dW.shape[1]), []
    for r in range(full):
        lo, hi = (v * unit for v in _own(n, full, r))
        if lo < mine.shape[1]:
            t = dW.new_zeros(blocks, hi - lo, dW.shape[1])
            part = mine[:, lo:hi]
            t[:, : part.shape[1]] = part
            out.append(t.view(-1, dW.shape[1]))
    return out


def exact(case, seed):
    kind = case["kind"]
    if kind in ("reshard", "mapped"):
        return None  # copies
    s = prepare(case, seed)
    if kind == "mlp":
        return _mlp64(s["mlp"])
    if kind == "attn":
        return _attn64(case, s["attn"])
    if kind == "core":
        q, kv = case["heads"], case["kv"]
        C, LSE, dQKV = _core64(case["n_seq"], case["seq"], q, kv, [j // (q // kv) for j in range(q)], case["dim"], case["causal"], _d(s["QKV"]),
                               None if s["dC"] is None else _d(s["dC"]))
        return dict(C=C, LSE=LSE, dQKV=dQKV) if case["back"] else dict(C=C, LSE=LSE)
    a, m = _attn64(case, s["attn"]), _mlp64(s["mlp"])
    d, full = case["dim"], case["full"]
    grads = [_full_shards(a["dWqkv"], 3, d, case["n_q"], full), _full_shards(a["dWo"], 1, d, case["n_q"], full),
             _full_shards(m["dA"], 1, 1, case["ffn"], full), _full_shards(m["dB"], 1, 1, case["ffn"], full)]
    return dict(Zattn=a["Z"], Zmlp=m["Z"][0], dXmlp=m["dX"][0], dXattn=a["dX"], C=a["C"], dQKV=a["dQKV"], grads=grads)
