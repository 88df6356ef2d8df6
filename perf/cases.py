"""The work a user of this library has it do: what is timed, on which inputs, and how closely
two correct implementations of it agree.

A case is one step of a pipeline stage through the public entry points (the Python binding of
include/gpt_stage.h and the schedules of harness.py), or one attention operator alone:

  step       for every micro-batch gpt_stage_fwd then gpt_stage_bwd on one stream
  decoupled  all forwards on a forward stream, all backward data phases on a backward stream,
             then one weight phase over the micro-batches
  forward    the forward phase alone (the forward instance of a decoupled pair, evaluation)
  backward   the backward phase alone on a stash written before (the backward instance)
  traversal  several model chunks x micro-batches through gpt_dpp_run, breadth first, one weight
             phase per chunk
  attention  gpt_stage_op_attention_fwd then gpt_stage_op_attention_bwd

Gradients are accumulated by the library, so a step begins by zeroing them, and weight images
(`prepare`) are rebuilt in every step that uses them: the weights change once per step.
"""
import torch

from paper_2507_19845_amd import binding as B
from paper_2507_19845_amd import harness, synth


def _stage(name, path, dtype, layers, hidden, heads, head_dim, ffn, seq, batch, microbatches=1, gelu="tanh",
           recompute=0, fp16=False, images=False, chunks=1, out_std=0.02):
    return {"name": name, "path": path, "dtype": dtype, "layers": layers, "hidden": hidden, "heads": heads,
            "head_dim": head_dim, "ffn": ffn, "seq": seq, "batch": batch, "microbatches": microbatches, "gelu": gelu,
            "recompute": recompute, "fp16": fp16, "images": images, "chunks": chunks, "out_std": out_std}


def listed():
    return [
        # smoke tests and parity checks of a schedule: a handful of microseconds of work per
        # kernel, everything is launches and latency (the `tiny_fp32` workload)
        _stage("tiny_fp32", "step", "fp32", 1, 128, 4, 32, 512, 64, 2),
        # an fp32 reference run of a small model on sequences of an odd length
        _stage("small_fp32_odd", "step", "fp32", 2, 512, 8, 64, 2048, 333, 3, gelu="erf"),
        # a small bf16 stage whose widths divide into no tile size evenly, two micro-batches
        _stage("small_bf16_odd", "step", "bf16", 2, 320, 5, 64, 832, 192, 2, microbatches=2, gelu="erf"),
        # one step of a medium model on one micro-batch (`gpt_medium_bf16`)
        _stage("medium_bf16", "step", "bf16", 4, 1024, 16, 64, 4096, 1024, 4),
        # a pipeline stage of a 13B-parameter model, one sequence per micro-batch (`gpt13b_bf16`)
        _stage("13b_bf16", "step", "bf16", 2, 5120, 40, 128, 20480, 2048, 1, out_std=0.01),
        # the breadth-first decoupled schedule over eight micro-batches (`decoupled_bf16`, the
        # benchmark's default), weight images rebuilt per step
        _stage("decoupled_bf16", "decoupled", "bf16", 4, 4096, 32, 128, 16384, 4096, 1, microbatches=8, images=True),
        # one tensor-parallel share of a 175B-parameter model with fp16 forward activations
        # (`tp_share_175b_bf16`); the fp16 forward reads the weights through images
        _stage("tp_share_175b", "step", "bf16", 2, 12288, 12, 128, 6144, 2048, 1, fp16=True, images=True),
        # the forward instance of a decoupled pair (also: evaluation) on a sequence length that is
        # not a multiple of the tile sizes
        _stage("forward_only", "forward", "bf16", 2, 2048, 16, 128, 8192, 1984, 2),
        # the backward instance of a decoupled pair that keeps a third less stash
        _stage("backward_recompute", "backward", "bf16", 2, 2048, 16, 128, 8192, 2048, 1, recompute=1),
        # four chunks of a small model traversed breadth first over eight small micro-batches
        _stage("traversal", "traversal", "bf16", 1, 1024, 16, 64, 4096, 512, 1, microbatches=8, chunks=4),
        # long-context attention alone, an odd length
        _stage("attention_long", "attention", "bf16", 1, 2048, 16, 128, 0, 8191, 1),
        # attention of many short sequences with narrow heads
        _stage("attention_short", "attention", "bf16", 1, 384, 12, 32, 0, 333, 16),
    ]


def _log_uniform(rng, lo, hi, step):
    """A multiple of `step` between lo and hi, spread over the logarithm."""
    v = lo * (hi / lo) ** rng.random()
    return max(step, int(round(v / step)) * step)


def _draw_once(rng):
    path = rng.choice(["step", "step", "step", "decoupled", "forward", "backward", "traversal", "attention"])
    gelu = rng.choice(["tanh", "tanh", "erf"])
    if path == "attention":
        d = rng.choice([32, 64, 128])
        seq = _log_uniform(rng, 64, 8192, 1)
        heads = _log_uniform(rng, 2, 32, 1)
        batch = max(1, min(16, _log_uniform(rng, 1, 16, 1), 32768 // seq))
        return _stage("", path, "bf16", 1, heads * d, heads, d, 0, seq, batch)
    if path == "step" and rng.random() < 0.35:       # fp32 stages: reference runs of small models
        d = rng.choice([32, 64, 128])
        heads = _log_uniform(rng, 1, 512 // d, 1)
        hidden = heads * d if rng.random() < 0.7 else _log_uniform(rng, 128, 512, 8)
        return _stage("", path, "fp32", rng.choice([1, 2]), hidden, heads, d, _log_uniform(rng, 2 * hidden, 4 * hidden, 8),
                      _log_uniform(rng, 33, 512, 1), rng.choice([1, 2, 3]), gelu=gelu)
    d = rng.choice([64, 128, 128])
    hidden = _log_uniform(rng, 256, 6144, d)
    heads = hidden // d if rng.random() < 0.75 else max(1, hidden // d // rng.choice([2, 4]))
    ffn = _log_uniform(rng, 2 * hidden, 4 * hidden, 64)
    batch = rng.choice([1, 1, 2, 4])
    seq = min(4096, _log_uniform(rng, 128, 4096, 64), max(128, 8192 // batch // 64 * 64))
    layers, microbatches, chunks, recompute, fp16 = rng.choice([1, 2]), 1, 1, 0, False
    if path == "step":
        microbatches = rng.choice([1, 1, 2])
        recompute = rng.choice([0, 0, 0, 1, 2])
        fp16 = d == 128 and rng.random() < 0.3
        if fp16:
            ffn, hidden = (ffn + 127) // 128 * 128, (hidden + 127) // 128 * 128
    elif path == "decoupled":
        microbatches = rng.choice([2, 3, 4, 8])
    elif path == "backward":
        recompute = rng.choice([0, 1, 2])
    elif path == "traversal":
        layers, microbatches, chunks = 1, rng.choice([2, 4, 8]), rng.choice([2, 4])
    return _stage("", path, "bf16", layers, hidden, heads, d, ffn, seq, batch, microbatches, gelu, recompute, fp16,
                  images=fp16 or (path == "decoupled" and microbatches >= 3), chunks=chunks)


def draw(rng):
    while True:
        case = _draw_once(rng)
        if work(case)["flops"] <= 2e13:      # a tenth of the largest listed case
            del case["name"]
            return case


def _shape(case):
    return synth.StageShape("case", n_layers=case["layers"], hidden=case["hidden"], n_heads=case["heads"],
                            head_dim=case["head_dim"], ffn=case["ffn"], seq=case["seq"], batch=case["batch"],
                            dtype=case["dtype"], n_microbatches=case["microbatches"], gelu=case["gelu"],
                            recompute=case["recompute"], fwd_fp16=case["fp16"])


def _fill_weights(w, cfg, case, gen):
    """Weights N(0, 0.02) (output projections N(0, out_std)), small biases, LayerNorm scales
    around 1: what a stage holds early in training."""
    for layer in range(cfg.n_layers):
        for tid, name in enumerate(synth.TENSOR_NAMES):
            off, n = B.gpt_stage_param_offset(cfg, layer, tid)
            t = w[off:off + n]
            if name.startswith("ln"):
                t.normal_(1.0 if name.endswith("_g") else 0.0, 0.1, generator=gen)
            else:
                t.normal_(0.0, case["out_std"] if name in ("w_o", "w_fc2") else 0.02, generator=gen)


class _State:
    """What a user's program keeps: buffers, weights, inputs, output tensors."""


def prepare(case, seed):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    s = _State()
    s.case = case
    n_mb = case["microbatches"]
    tdt = torch.bfloat16 if case["dtype"] == "bf16" else torch.float32

    def normal(*shape):
        return torch.empty(shape, dtype=tdt, device="cuda").normal_(generator=gen)

    if case["path"] == "attention":
        Bt, S, a, d = case["batch"], case["seq"], case["heads"], case["head_dim"]
        s.dt = B.GPTS_BF16 if case["dtype"] == "bf16" else B.GPTS_FP32
        s.qkv, s.dout = normal(Bt, S, 3 * a * d), normal(Bt, S, a * d)
        s.out, s.dqkv = torch.empty_like(s.dout), torch.empty_like(s.qkv)
        s.lse = torch.empty((Bt, a, S), dtype=torch.float32, device="cuda")
        s.scratch = [torch.empty(max(B.gpt_stage_op_attention_scratch_bytes(s.dt, Bt, S, a, d, ph), 256),
                                 dtype=torch.uint8, device="cuda") for ph in (0, 1)]
        return s

    shape = _shape(case)
    s.xs = [normal(shape.batch, shape.seq, shape.hidden) for _ in range(n_mb)]
    s.dys = [normal(shape.batch, shape.seq, shape.hidden) for _ in range(n_mb)]
    s.ys = [torch.empty_like(x) for x in s.xs]
    s.dxs = [torch.empty_like(x) for x in s.xs]
    if case["path"] == "traversal":
        cfg = B.make_cfg(shape)
        n = B.gpt_stage_param_count(cfg)
        s.ws = torch.empty(B.gpt_stage_workspace_bytes(cfg, 1), dtype=torch.uint8, device="cuda")
        s.weights = [torch.empty(n, dtype=tdt, device="cuda") for _ in range(case["chunks"])]
        for w in s.weights:
            _fill_weights(w, cfg, case, gen)
        s.dparams = [torch.zeros(n, dtype=torch.float32, device="cuda") for _ in range(case["chunks"])]
        s.chunks = [B.make_params(cfg, w, s.ws) for w in s.weights]
        s.stash = torch.empty(B.gpt_dpp_stash_slot_bytes(s.chunks) * case["chunks"] * n_mb, dtype=torch.uint8, device="cuda")
        s.act = torch.empty(B.gpt_dpp_act_slot_bytes(cfg) * (n_mb + 2), dtype=torch.uint8, device="cuda")
        s.grad_pool = torch.empty(B.gpt_dpp_grad_slot_bytes(s.chunks) * n_mb, dtype=torch.uint8, device="cuda")
        return s

    s.bufs = B.StageBuffers(shape, n_stash=n_mb if case["path"] == "decoupled" else 1)
    _fill_weights(s.bufs.weights, s.bufs.cfg, case, gen)
    if case["path"] == "decoupled":
        s.bufs.alloc_grad_stash(n_mb)
    if case["images"]:
        s.bufs.prepare()
    s.runner = harness.StageRunner(s.bufs)
    if case["path"] == "backward":
        B.gpt_stage_fwd(s.bufs.params(), s.xs[0], s.bufs.stash[0], s.ys[0])
    return s


def run(state):
    s, case = state, state.case
    path = case["path"]
    if path == "attention":
        Bt, S, a, d = case["batch"], case["seq"], case["heads"], case["head_dim"]
        B.gpt_stage_op_attention_fwd(s.dt, Bt, S, a, d, s.qkv, s.out, s.lse, s.scratch[0])
        B.gpt_stage_op_attention_bwd(s.dt, Bt, S, a, d, s.qkv, s.out, s.lse, s.dout, s.dqkv, s.scratch[1])
        return [s.out, s.lse, s.dqkv]
    if path == "traversal":
        for g in s.dparams:
            g.zero_()
        B.gpt_dpp_run(B.GPT_DPP_BFC, s.chunks, s.xs, s.dys, s.ys, s.dxs, s.dparams, s.stash, s.act, grad_pool=s.grad_pool)
        return s.ys + s.dxs + s.dparams
    b = s.bufs
    if path == "forward":
        B.gpt_stage_fwd(b.params(), s.xs[0], b.stash[0], s.ys[0])
        return s.ys
    b.dparams.zero_()
    if path == "backward":
        B.gpt_stage_bwd(b.params(), b.stash[0], s.dys[0], s.dxs[0], b.dparams)
        return s.dxs + [b.dparams]
    if case["images"]:
        b.prepare()
    if path == "decoupled":
        s.runner.decoupled(s.xs, s.dys, s.ys, s.dxs, split_wgrad=True)
    else:
        s.runner.coupled(s.xs, s.dys, s.ys, s.dxs)
    return s.ys + s.dxs + [b.dparams]


def work(case):
    """Multiply-adds of the linears and of the causal half of attention (recomputation not
    counted); every input read once and every output written once."""
    L, H, F, S, a, d = (case[k] for k in ("layers", "hidden", "ffn", "seq", "heads", "head_dim"))
    T, P, e = case["batch"] * S, a * d, 2 if case["dtype"] == "bf16" else 4
    attn = 4.0 * case["batch"] * a * d * S * (S + 1) / 2
    if case["path"] == "attention":
        # q, k, v, dO in; out, lse, dq, dk, dv out
        return {"flops": 3 * attn, "bytes": 8.0 * T * P * e + 4.0 * case["batch"] * a * S}
    n_mb, chunks = case["microbatches"], case["chunks"]
    fwd = chunks * n_mb * L * (2.0 * T * (4.0 * P * H + 2.0 * H * F) + attn)
    params = chunks * L * (4.0 * P * H + 2.0 * H * F + 5.0 * H + F + 3.0 * P + H)
    act = float(n_mb) * T * H * e
    # what one micro-batch's stash has to hold per layer when only the layer's input is kept
    stash = float(L) * T * H * 4
    if case["path"] == "forward":
        return {"flops": fwd, "bytes": params * e + 2 * act + stash}
    if case["path"] == "backward":
        return {"flops": 2 * fwd, "bytes": params * (e + 4) + 2 * act + stash}
    return {"flops": 3 * fwd, "bytes": params * (e + 4) + 4 * act}


def _attention64(qkv, heads, d):
    """Causal softmax attention and its log-sum-exp, in 64 bits, one head at a time.
    qkv [S, 3*heads*d] with rows [Q heads | K heads | V heads]."""
    S, P = qkv.shape[0], heads * d
    masked = torch.ones(S, S, dtype=torch.bool, device=qkv.device).triu(1)
    outs, lses = [], []
    for n in range(heads):
        q, k, v = (qkv[:, i * P + n * d:i * P + (n + 1) * d] for i in range(3))
        s = (q @ k.t() / d ** 0.5).masked_fill(masked, float("-inf"))
        outs.append(torch.softmax(s, dim=-1) @ v)
        lses.append(torch.logsumexp(s.detach(), dim=-1))
    return torch.cat(outs, dim=1), torch.stack(lses)


def _layer64(x, p, case):
    """One decoder layer in 64 bits; x [batch, seq, hidden], p the layer's twelve tensors."""
    F = torch.nn.functional
    Bt, S, H = x.shape
    g1, b1, wqkv, bqkv, wo, bo, g2, b2, w1, c1, w2, c2 = p
    qkv = F.linear(F.layer_norm(x, (H,), g1, b1, 1e-5), wqkv, bqkv)
    c = torch.stack([_attention64(qkv[b], case["heads"], case["head_dim"])[0] for b in range(Bt)])
    x1 = x + F.linear(c, wo, bo)
    u = F.linear(F.layer_norm(x1, (H,), g2, b2, 1e-5), w1, c1)
    return x1 + F.linear(F.gelu(u, approximate="tanh" if case["gelu"] == "tanh" else "none"), w2, c2)


def exact(case, seed):
    """The outputs of run() from torch's 64-bit operators and autograd on the same inputs.  The
    flat parameter buffer holds, layer by layer, ln1_g, ln1_b, w_qkv, b_qkv, w_o, b_o, ln2_g,
    ln2_b, w_fc1, b_fc1, w_fc2, b_fc2 without gaps."""
    s = prepare(case, seed)
    if case["path"] == "attention":
        a, d = case["heads"], case["head_dim"]
        outs, lses, grads = [], [], []
        for b in range(case["batch"]):
            qkv = s.qkv[b].double().requires_grad_()
            out, lse = _attention64(qkv, a, d)
            out.backward(s.dout[b].double())
            outs.append(out.detach())
            lses.append(lse)
            grads.append(qkv.grad)
        return [torch.stack(outs), torch.stack(lses), torch.stack(grads)]
    xs, dys = s.xs, s.dys
    weights = s.weights if case["path"] == "traversal" else [s.bufs.weights]
    weights = [w.double() for w in weights]
    del s                                    # the stage's own buffers are not needed
    H, P, F = case["hidden"], case["heads"] * case["head_dim"], case["ffn"]
    shapes = [(H,), (H,), (3 * P, H), (3 * P,), (H, P), (H,), (H,), (H,), (F, H), (F,), (H, F), (H,)]
    chunks, grads = [], []
    for w in weights:
        g, layers, off = torch.zeros_like(w), [], 0
        for _ in range(case["layers"]):
            layer = []
            for shape in shapes:
                n = 1
                for size in shape:
                    n *= size
                t = w[off:off + n].view(shape).requires_grad_()
                t.grad = g[off:off + n].view(shape)      # micro-batches add up in place
                layer.append(t)
                off += n
            layers.append(layer)
        chunks.append(layers)
        grads.append(g)
    ys, dxs = [], []
    for x, dy in zip(xs, dys):
        x = x.double().requires_grad_()
        y = x
        for layers in chunks:
            for layer in layers:
                y = _layer64(y, layer, case)
        if case["path"] != "forward":
            y.backward(dy.double())
            dxs.append(x.grad)
        ys.append(y.detach())
        del x, y
    if case["path"] == "forward":
        return ys
    if case["path"] == "backward":
        return dxs + grads
    return ys + dxs + grads


def tolerance(case):
    """Relative error in the 2-norm, and the largest single difference over the tensor's root mean
    square (or the value, where larger): about four times what these cases show against the same
    stage computed in 64 bits.  Measured: fp32 stages up to 7.7e-7 and 5.7e-6 (weight gradients);
    bf16 stages up to 5.2e-3 and 7e-2 (four layers), attention alone up to 3.2e-3 and 0.15 (the
    gradients of keys that many queries share)."""
    if case["dtype"] == "fp32":
        return {"rel": 4e-6, "max": 5e-5}
    return {"rel": 1.2e-2 if case["path"] == "attention" else 2e-2, "max": 0.5}
