"""GPU parity: the HIP library, called through its C-ABI, against the CPU fp64
oracle on the same seeded inputs, tensor by tensor.  Tolerance (tensor-max-
normalised max error): 1e-4 for fp32 stages, 2e-2 for bf16 stages."""
import numpy as np
import pytest
import torch

from oracle import gpt_stage_oracle as orc
from paper_2507_19845_amd import binding as B
from paper_2507_19845_amd import synth

from parity_util import TOL, compare, gpu_run, max_norm_err, oracle_run, p64

pytestmark = pytest.mark.gpu

W = synth.WORKLOADS


def _inputs(shape, n_mb=1, seed=0):
    params = synth.make_params(shape, seed)
    xs = [synth.make_x(shape, seed, m) for m in range(n_mb)]
    dys = [synth.make_dy(shape, seed, m) for m in range(n_mb)]
    return params, xs, dys


def _report(name, errs):
    worst = max(errs, key=errs.get)
    print(f"[parity] {name}: worst {worst} = {errs[worst]:.3e}", flush=True)


# ------------------------------------------------------------- whole stage ----
SMALL = [
    W[0],                                                        # workload 1 as specified (fp32)
    W[0].with_(name="tiny_fp32_erf", gelu="erf", bias_std=0.02, ln_jitter=0.1),
    W[0].with_(name="tiny_fp32_ragged", seq=50, batch=3, n_layers=2, bias_std=0.02, ln_jitter=0.1),
    W[0].with_(name="tiny_fp32_seq1", seq=1, batch=5),
    W[0].with_(name="tiny_fp32_tp", hidden=192, n_heads=2, head_dim=32, ffn=136, bias_std=0.02),
    W[0].with_(name="tiny_fp32_d64", n_heads=2, head_dim=64, seq=70),
    W[0].with_(name="tiny_fp32_d128", n_heads=1, head_dim=128, seq=33),
    # bf16 cases spanning several tiles with a ragged (non-256) tail in every dimension
    W[1].with_(name="bf16_small", n_layers=2, hidden=320, n_heads=5, head_dim=64, ffn=832, seq=192,
               batch=2, bias_std=0.02, ln_jitter=0.1),
    W[1].with_(name="bf16_d128_tp", n_layers=2, hidden=512, n_heads=3, head_dim=128, ffn=448,
               seq=320, batch=1, bias_std=0.02, ln_jitter=0.1),
    W[1].with_(name="bf16_erf", n_layers=1, hidden=256, n_heads=4, head_dim=64, ffn=512, seq=64,
               batch=1, gelu="erf", bias_std=0.02),
    # bf16 heads of dimension 32 (matrix-core attention with 4-chunk tile rows)
    W[1].with_(name="bf16_d32", n_layers=2, hidden=256, n_heads=6, head_dim=32, ffn=512, seq=320,
               batch=1, bias_std=0.02, ln_jitter=0.1),
    # fp16 forward activations (cfg.fwd_fp16): ragged token count against the 256-row tiles,
    # attention width != hidden, both head dimensions, both GeLU forms
    W[1].with_(name="bf16_fwd16_d128", n_layers=2, hidden=512, n_heads=3, head_dim=128, ffn=640,
               seq=320, batch=1, bias_std=0.02, ln_jitter=0.1, fwd_fp16=True),
    W[1].with_(name="bf16_fwd16_d32", n_layers=1, hidden=256, n_heads=4, head_dim=32, ffn=512,
               seq=200 + 56, batch=1, bias_std=0.02, ln_jitter=0.1, fwd_fp16=True),
    W[1].with_(name="bf16_fwd16_d64_erf", n_layers=2, hidden=384, n_heads=4, head_dim=64, ffn=896,
               seq=192, batch=2, gelu="erf", bias_std=0.02, ln_jitter=0.1, fwd_fp16=True),
    # the same with so many heads times sequences that attention takes its form of one wave per 32 rows in
    # forward and one launch in backward (800 and 1280 blocks of 64 rows; one wave per 32 rows at head dimensions 32
    # and 64), then, in the "many" shapes (over 1700 blocks), a launch for each side; the last block short
    W[1].with_(name="bf16_fwd16_d128_full_chip", n_layers=1, hidden=256, n_heads=10, head_dim=128, ffn=256,
               seq=260, batch=16, bias_std=0.02, ln_jitter=0.1, fwd_fp16=True),
    W[1].with_(name="bf16_fwd16_d128_many", n_layers=1, hidden=128, n_heads=10, head_dim=128, ffn=128,
               seq=260, batch=48, bias_std=0.02, ln_jitter=0.1, fwd_fp16=True),
    W[1].with_(name="bf16_fwd16_d64_many", n_layers=1, hidden=128, n_heads=10, head_dim=64, ffn=128,
               seq=260, batch=48, bias_std=0.02, ln_jitter=0.1, fwd_fp16=True),
    W[1].with_(name="bf16_fwd16_d32_many", n_layers=1, hidden=128, n_heads=12, head_dim=32, ffn=128,
               seq=260, batch=32, bias_std=0.02, ln_jitter=0.1, fwd_fp16=True),
    W[1].with_(name="bf16_fwd16_d64_full_chip", n_layers=1, hidden=256, n_heads=10, head_dim=64, ffn=256,
               seq=260, batch=16, bias_std=0.02, ln_jitter=0.1, fwd_fp16=True),
    W[1].with_(name="bf16_fwd16_d32_full_chip", n_layers=1, hidden=256, n_heads=16, head_dim=32, ffn=256,
               seq=260, batch=16, bias_std=0.02, ln_jitter=0.1, fwd_fp16=True),
]


@pytest.mark.parametrize("shape", SMALL, ids=lambda s: s.name)
def test_stage_matches_oracle(shape):
    print(f"[case] stage {shape}", flush=True)
    params, xs, dys = _inputs(shape)
    got = gpu_run(shape, params, xs, dys)
    ref = oracle_run(shape, params, xs, dys)
    _report(shape.name, compare(shape, got, ref))


def test_microbatch_accumulation_and_decoupled_schedule():
    """3 micro-batches: gradients accumulate across calls; the decoupled
    (all-forward-then-all-backward, two streams) schedule gives bit-identical
    results to the coupled one; both match the oracle."""
    shape = W[1].with_(name="bf16_mb", n_layers=2, hidden=256, n_heads=4, head_dim=64, ffn=512,
                       seq=128, batch=1, bias_std=0.02, ln_jitter=0.1)
    print(f"[case] microbatches {shape}", flush=True)
    params, xs, dys = _inputs(shape, n_mb=3)
    a = gpu_run(shape, params, xs, dys, decoupled=False)
    b = gpu_run(shape, params, xs, dys, decoupled=True)
    for i in range(3):
        assert np.array_equal(a[0][i], b[0][i]) and np.array_equal(a[1][i], b[1][i])
    for ga, gb in zip(a[2], b[2]):
        for k in ga:
            assert np.array_equal(ga[k], gb[k]), k
    _report(shape.name, compare(shape, b, oracle_run(shape, params, xs, dys)))


@pytest.mark.parametrize("mode", ["full_stash", "recompute", "fwd_fp16"])
def test_split_backward_data_phase_then_one_weight_phase(mode):
    """gpt_stage_bwd_data_only for every micro-batch, then gpt_stage_wgrad_flush once.
    y, dx, bias and LayerNorm gradients must equal the unsplit decoupled run bit for bit
    (same kernels).  Weight gradients: with a full stash the qkv, fc1 and fc2 products here
    contract over all three micro-batches in one launch (>= 100 tiles of 256x256), which
    changes the fp32 summation order only; out-proj (64 tiles) and the modes whose stash
    lacks the activations take one product per micro-batch and stay bit-identical.
    Everything against the oracle as well."""
    shape = W[1].with_(name=f"bf16_split_{mode}", n_layers=2, hidden=2048, n_heads=16, head_dim=128, ffn=4096,
                       seq=256, batch=1, bias_std=0.02, ln_jitter=0.1, recompute=mode == "recompute",
                       fwd_fp16=mode == "fwd_fp16")
    print(f"[case] split backward {shape}", flush=True)
    params, xs, dys = _inputs(shape, n_mb=3)
    whole = gpu_run(shape, params, xs, dys, decoupled=True)
    split = gpu_run(shape, params, xs, dys, decoupled=True, split_wgrad=True)
    for i in range(3):
        assert np.array_equal(whole[0][i], split[0][i]) and np.array_equal(whole[1][i], split[1][i])
    one_launch = ("w_qkv", "w_fc1", "w_fc2") if mode == "full_stash" else ()
    for ga, gb in zip(whole[2], split[2]):
        for k in ga:
            if k in one_launch:
                assert not np.array_equal(ga[k], gb[k]), f"{k}: expected the one-launch path"
                assert max_norm_err(gb[k], ga[k]) < 2e-6, k
            else:
                assert np.array_equal(ga[k], gb[k]), k
    _report(shape.name, compare(shape, split, oracle_run(shape, params, xs, dys)))


@pytest.mark.parametrize("n_mb,seq,hidden,heads,ffn", [(4, 64, 128, 1, 256), (5, 192, 192, 5, 2112), (4, 320, 448, 2, 2112),
                                                       (5, 64, 832, 3, 2112), (5, 320, 832, 5, 2112),
                                                       (4, 64, 2112, 5, 4160), (5, 192, 2560, 2, 5056),
                                                       (4, 192, 960, 16, 2112), (4, 192, 1024, 16, 2112),
                                                       (4, 192, 1728, 5, 2752), (5, 192, 1472, 16, 3200)],
                         ids=["64x32", "128x64", "128x128", "128x128_short", "128x128_five", "256x128_shared",
                              "256x128_shared_five", "192x192", "256x160", "256x192", "256x256"])
def test_split_backward_four_or_more_microbatches(n_mb, seq, hidden, heads, ffn):
    """From four micro-batches on the weight phase contracts over all of them in one launch, whatever the
    widths: each tile of the products, segments of one, three and five slices of 64 (shorter than the
    ring of stages, odd) and the tiles with slices of 32.  The fp32 summation order changes and
    nothing else: at most 1600 tokens, so up to sqrt(1600) roundings of 2^-24, 2.4e-6, of the largest sum.  The
    same bits from one launch per linear (which a tracer asks for); micro-batches that are not equally
    spaced take one product each and keep the bits of the unsplit run."""
    shape = W[1].with_(name="bf16_split_many", n_layers=1, hidden=hidden, n_heads=heads, head_dim=64, ffn=ffn, seq=seq,
                       batch=1, bias_std=0.02, ln_jitter=0.1)
    print(f"[case] split backward, {n_mb} micro-batches {shape}", flush=True)
    params, xs, dys = _inputs(shape, n_mb=n_mb)
    whole = gpu_run(shape, params, xs, dys, decoupled=True)
    split = gpu_run(shape, params, xs, dys, decoupled=True, split_wgrad=True)
    for a, b in zip(whole[0] + whole[1], split[0] + split[1]):
        assert np.array_equal(a, b)
    for k, a in whole[2][0].items():
        b = split[2][0][k]
        if k.startswith("w_"):
            assert not np.array_equal(a, b), f"{k}: expected the one-launch path"
            assert max_norm_err(b, a) < 2.4e-6, k
        else:
            assert np.array_equal(a, b), k
    tr = B.gpt_stage_trace_create(64 * n_mb)
    try:
        traced = gpu_run(shape, params, xs, dys, decoupled=True, split_wgrad=True, trace=tr)
        recs, _ = B.gpt_stage_trace_collect(tr, 64 * n_mb)
    finally:
        B.gpt_stage_trace_destroy(tr)
    assert len([r for r in recs if r["op"] == "gemm_wgrad"]) == 4
    bufs = B.StageBuffers(shape, n_stash=n_mb + 1)
    bufs.load_params(params)
    del bufs.stash[1]                                    # a gap between the first two
    apart = gpu_run(shape, params, xs, dys, decoupled=True, split_wgrad=True, bufs=bufs)
    for k, a in whole[2][0].items():
        assert np.array_equal(split[2][0][k], traced[2][0][k]) and np.array_equal(a, apart[2][0][k]), k
    if hidden <= 832:
        _report(shape.name, compare(shape, split, oracle_run(shape, params, xs, dys)))


def test_split_backward_other_paths():
    """The weight phase of fewer than four micro-batches where the segments are not whole multiples of 128
    tokens: one accumulating product per micro-batch, bit-identical to the unsplit run; and a single
    micro-batch (one product, nothing to concatenate)."""
    shape = W[1].with_(name="bf16_split_192", n_layers=2, hidden=2048, n_heads=16, head_dim=128, ffn=4096,
                       seq=192, batch=1, bias_std=0.02, ln_jitter=0.1)
    print(f"[case] split backward, fallback paths {shape}", flush=True)
    params, xs, dys = _inputs(shape, n_mb=2)
    whole = gpu_run(shape, params, xs, dys, decoupled=True)
    split = gpu_run(shape, params, xs, dys, decoupled=True, split_wgrad=True)
    for a, b in zip(whole[0] + whole[1], split[0] + split[1]):
        assert np.array_equal(a, b)
    for ga, gb in zip(whole[2], split[2]):
        for k in ga:
            assert np.array_equal(ga[k], gb[k]), k
    one = shape.with_(name="bf16_split_one", seq=256)
    params, xs, dys = _inputs(one, n_mb=1)
    whole = gpu_run(one, params, xs, dys, decoupled=True)
    split = gpu_run(one, params, xs, dys, decoupled=True, split_wgrad=True)
    assert np.array_equal(whole[0][0], split[0][0]) and np.array_equal(whole[1][0], split[1][0])
    for ga, gb in zip(whole[2], split[2]):
        for k in ga:
            assert np.array_equal(ga[k], gb[k]), k     # one segment: the same product, the same bits
    _report(one.name, compare(one, split, oracle_run(one, params, xs, dys)))


def test_backward_stream_waits_for_the_forward_event():
    """The forward stream is held back by a long spin kernel; the backward stream
    must still see a complete stash because bwd_only waits on the event that the
    last fwd_only records.  Without that wait it would read the zero-filled stash."""
    from paper_2507_19845_amd import harness
    shape = W[1].with_(name="bf16_evt", n_layers=1, hidden=256, n_heads=4, head_dim=64, ffn=512,
                       seq=128, batch=1, bias_std=0.02)
    print(f"[case] event plumbing {shape}", flush=True)
    params, xs, dys = _inputs(shape, n_mb=2)
    ref = gpu_run(shape, params, xs, dys, decoupled=False)
    bufs = B.StageBuffers(shape, n_stash=2)
    bufs.load_params(params)
    for s_ in bufs.stash:
        s_.zero_()
    xd = [B.to_device(x, shape.dtype) for x in xs]
    dyd = [B.to_device(d, shape.dtype) for d in dys]
    ys, dxs = [bufs.act() for _ in xs], [bufs.act() for _ in xs]
    runner = harness.StageRunner(bufs)
    torch.cuda.synchronize()
    with torch.cuda.stream(runner.fwd_stream):
        torch.cuda._sleep(400_000_000)          # ~0.2 s of spinning ahead of the forwards
    runner.decoupled(xd, dyd, ys, dxs)
    torch.cuda.synchronize()
    for i in range(2):
        assert np.array_equal(B.to_host(ys[i]), ref[0][i])
        assert np.array_equal(B.to_host(dxs[i]), ref[1][i])
    for ga, gb in zip(bufs.read_grads(), ref[2]):
        for k in ga:
            assert np.array_equal(ga[k], gb[k]), k


@pytest.mark.parametrize("ffn", [16384 - 64, 8192], ids=["ffn_ragged", "ffn_mult_128"])
def test_prepared_weights_give_identical_results(ffn):
    """With the weight images of gpt_stage_prepare() the forward products read the same
    numbers through a different layout: every output must be bit-identical to the run on the
    raw weights.  One layer of the decoupled workload's shape, all 256x256 tiles.  ffn 16320: an
    image whose last tile of 256 rows is short, and a contraction of an odd number of slices; ffn 8192:
    whole tiles, as in the benchmark."""
    shape = W[3].with_(name="bf16_prepared", n_layers=1, ffn=ffn, n_microbatches=1, bias_std=0.02)
    _check_prepared_weights(shape)


@pytest.mark.parametrize("seq,hidden,ffn", [(1984, 5056, 320), (1984, 4160, 320), (1984, 1088, 6080), (448, 832, 3008)],
                         ids=["256x160", "192x192", "256x192", "128x64_64x32"])
def test_prepared_weights_give_identical_results_in_every_tile(seq, hidden, ffn):
    """The same with tiles that do not divide the image's tiles of 256 rows, or are smaller, and widths that
    leave the last tile of both short: 256x160 and 64x64; 192x192; 256x192, 256x128 and 128x128; 128x64
    and 64x32."""
    heads, d = (5, 64) if seq == 448 else (1, 128)
    _check_prepared_weights(W[1].with_(name="bf16_prepared_tiles", n_layers=1, hidden=hidden, n_heads=heads, head_dim=d,
                                       ffn=ffn, seq=seq, batch=1, bias_std=0.02))


def _check_prepared_weights(shape):
    print(f"[case] prepared weights {shape}", flush=True)
    params, xs, dys = _inputs(shape)
    bufs = B.StageBuffers(shape)
    bufs.load_params(params)
    raw = gpu_run(shape, params, xs, dys, bufs=bufs)
    assert B.gpt_stage_prepared_bytes(bufs.cfg) > B.gpt_stage_param_bytes(bufs.cfg) * 0.99
    bufs.prepare()
    try:
        prep = gpu_run(shape, params, xs, dys, bufs=bufs)
    finally:
        bufs.unprepare()
    assert np.array_equal(raw[0][0], prep[0][0]) and np.array_equal(raw[1][0], prep[1][0])
    for ga, gb in zip(raw[2], prep[2]):
        for k in ga:
            assert np.array_equal(ga[k], gb[k]), k
    assert B.gpt_stage_prepared_bytes(B.make_cfg(W[0])) == 0      # fp32 stages have none


def test_operator_tracer_records_every_operator():
    """A traced forward+backward yields one record per operator in launch order with
    positive durations, leaves the results bit-identical, and exports as Chrome trace."""
    from paper_2507_19845_amd import harness
    shape = W[1].with_(name="bf16_trace", n_layers=2, hidden=256, n_heads=4, head_dim=64, ffn=512,
                       seq=128, batch=1)
    print(f"[case] tracer {shape}", flush=True)
    params, xs, dys = _inputs(shape)
    ref = gpu_run(shape, params, xs, dys)
    tr = B.gpt_stage_trace_create(64)
    got = gpu_run(shape, params, xs, dys, trace=tr)
    recs, dropped = B.gpt_stage_trace_collect(tr, 64)
    # per layer 7 forward and 13 backward operators (the out-proj and fc2 bias gradients ride on
    # the LayerNorm backward kernels), plus the top layer's fc2 bias gradient
    n_ops = 20 * shape.n_layers + 1
    assert dropped == 0 and len(recs) == n_ops
    assert [r["op"] for r in recs[:7]] == ["layernorm_fwd", "gemm_fwd", "attention_fwd", "gemm_fwd",
                                          "layernorm_fwd", "gemm_fwd", "gemm_fwd"]
    assert [r["phase"] for r in recs] == [0] * 14 + [1] * 27
    assert [r["layer"] for r in recs[14:]] == [1] * 14 + [0] * 13          # backward walks layers in reverse
    assert all(r["dur_ms"] > 0 for r in recs)
    assert all(b["start_ms"] >= a["start_ms"] for a, b in zip(recs, recs[1:]))
    T, H, F = shape.tokens, shape.hidden, shape.ffn
    assert recs[5]["flops"] == 2.0 * T * F * H                             # fc1 forward product
    assert np.array_equal(got[0][0], ref[0][0]) and np.array_equal(got[1][0], ref[1][0])
    doc = harness.chrome_trace(recs)
    assert len(doc["traceEvents"]) == len(recs) and doc["traceEvents"][1]["name"] == "gemm_fwd.qkv"
    # capacity overflow is counted, not fatal
    B.gpt_stage_trace_reset(tr)
    small = B.gpt_stage_trace_create(5)
    try:
        gpu_run(shape, params, xs, dys, trace=small)
        recs2, dropped2 = B.gpt_stage_trace_collect(small, 5)
    finally:
        B.gpt_stage_trace_destroy(small)
        B.gpt_stage_trace_destroy(tr)
    assert len(recs2) == 5 and dropped2 == n_ops - 5


@pytest.mark.parametrize("batch,hidden,ffn", [(97, 896, 2688), (130, 512, 2048), (3, 256, 512)])
def test_fc1_bias_gradient_needs_no_pass_over_du(batch, hidden, ffn):
    """The fc1 bias gradient comes out of the fc2 data gradient's epilogue however many rows of partial
    sums its tile makes of the tokens: 66 (192-row tiles of 6208 tokens), 88 and 6.  The operator
    that adds them up reads those rows and not dU.  Against the column sums of dU as stored: each of its
    values is rounded to bf16 (2^-9), the summed ones are not."""
    shape = W[1].with_(name="bf16_fc1_sums", n_layers=1, hidden=hidden, n_heads=1, head_dim=128, ffn=ffn, seq=64,
                       batch=batch)
    print(f"[case] fc1 bias sums {shape}", flush=True)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(batch)
    bufs = B.StageBuffers(shape)
    bufs.weights.normal_(0.0, 0.02, generator=gen)
    bufs.alloc_grad_stash(1)
    x, dy = (bufs.act().normal_(generator=gen) for _ in range(2))
    y, dx = bufs.act(), bufs.act()
    B.gpt_stage_fwd(bufs.params(), x, bufs.stash[0], y)
    tr = B.gpt_stage_trace_create(64)
    try:
        bufs.trace = tr
        B.gpt_stage_bwd_data_only(bufs.params(), bufs.stash[0], dy, dx, bufs.dparams, bufs.grad_stash[0])
        recs, _ = B.gpt_stage_trace_collect(tr, 64)
    finally:
        B.gpt_stage_trace_destroy(tr)
    T = shape.tokens
    fc1 = [r for r in recs if r["op"] == "bias_grad" and r["sub"] == 2]
    assert len(fc1) == 1 and fc1[0]["bytes"] <= T * ffn * 2 / 8      # dU itself is T * ffn * 2 bytes
    off = (T * hidden * 2 + 255) // 256 * 256                        # grad stash: dY, then dU, 256-byte aligned
    du = bufs.grad_stash[0][off:off + T * ffn * 2].view(torch.bfloat16).view(T, ffn).double()
    o, n = B.gpt_stage_param_offset(bufs.cfg, 0, synth.TENSOR_NAMES.index("b_fc1"))
    assert ((bufs.dparams[o:o + n].double() - du.sum(0)).abs() <= 2.0 ** -8 * du.abs().sum(0)).all()


def test_run_to_run_bitwise_determinism():
    shape = W[1].with_(name="bf16_det", n_layers=1, hidden=256, n_heads=4, head_dim=64, ffn=512,
                       seq=256, batch=2)
    print(f"[case] determinism {shape}", flush=True)
    params, xs, dys = _inputs(shape)
    a = gpu_run(shape, params, xs, dys)
    b = gpu_run(shape, params, xs, dys)
    assert np.array_equal(a[0][0], b[0][0]) and np.array_equal(a[1][0], b[1][0])
    for ga, gb in zip(a[2], b[2]):
        for k in ga:
            assert np.array_equal(ga[k], gb[k]), k


def test_zero_weight_identity_residual_on_gpu():
    """All W = 0, b = 0: y = x and dx = dy bit for bit; db_o = db_fc2 = sum_t dy."""
    shape = W[1].with_(name="bf16_zero", n_layers=2, hidden=256, n_heads=4, head_dim=64, ffn=512,
                       seq=128, batch=1)
    print(f"[case] zero weights {shape}", flush=True)
    params, xs, dys = _inputs(shape)
    for p in params:
        for k in p:
            if k[:2] in ("w_", "b_"):
                p[k][...] = 0.0
    ys, dxs, grads = gpu_run(shape, params, xs, dys)
    assert np.array_equal(ys[0], xs[0].astype(np.float64))
    assert np.array_equal(dxs[0], dys[0].astype(np.float64))
    colsum = dys[0].astype(np.float64).reshape(-1, shape.hidden).sum(0)
    for g in grads:
        for k, v in g.items():
            if k in ("b_o", "b_fc2"):
                assert max_norm_err(v, colsum) < 1e-5
            else:
                assert np.all(v == 0.0), k


def test_causality_on_gpu():
    shape = W[1].with_(name="bf16_causal", n_layers=2, hidden=256, n_heads=4, head_dim=64, ffn=512,
                       seq=192, batch=2)
    print(f"[case] causality {shape}", flush=True)
    params, xs, dys = _inputs(shape)
    y0, _, _ = gpu_run(shape, params, xs, dys)
    t = 100
    x2 = xs[0].copy()
    x2[0, t:, :] = synth.make_x(shape, 7)[0, t:, :]
    y1, _, _ = gpu_run(shape, params, [x2], dys)
    assert np.array_equal(y0[0][0, :t], y1[0][0, :t])
    assert np.array_equal(y0[0][1], y1[0][1])
    assert not np.array_equal(y0[0][0, t:], y1[0][0, t:])


# ------------------------------------------------------ full-size workloads ----
def test_workload2_full_size():
    shape = W[1]
    print(f"[case] full {shape}", flush=True)
    params, xs, dys = _inputs(shape)
    got = gpu_run(shape, params, xs, dys)
    ref = oracle_run(shape, params, xs, dys)
    _report(shape.name, compare(shape, got, ref))


def test_workload3_full_size():
    """13B-shaped stage at full size, every output tensor against the oracle."""
    shape = W[2]
    print(f"[case] full {shape}", flush=True)
    params, xs, dys = _inputs(shape)
    got = gpu_run(shape, params, xs, dys)
    ref = oracle_run(shape, params, xs, dys)
    _report(shape.name, compare(shape, got, ref))


def test_workload5_full_size():
    """One GPU's tensor-parallel share of a 175B-shaped layer at full size, every output
    tensor against the oracle at the bf16 bar.

    With N(0, 0.02) weights at hidden 12288 the attention logits have a standard deviation
    of ~4.9 (max ~23) and the softmax amplifies the rounding of every forward activation:
    with bf16 forward activations the gradients miss the bar by a factor of two (the CPU
    emulation in tests/test_rounding_emulation.py reproduces that with the oracle's own
    arithmetic and shows which tensors matter).  The workload therefore runs with
    cfg.fwd_fp16: forward activations in fp16, everything else bf16.  The same stage with
    bf16 forward activations is run too and must show the larger error, so that the
    switch is known to be what brings the workload inside the bar."""
    shape = W[4]
    assert shape.fwd_fp16
    print(f"[case] full {shape}", flush=True)
    params, xs, dys = _inputs(shape)
    got = gpu_run(shape, params, xs, dys)
    ref = oracle_run(shape, params, xs, dys)
    errs = compare(shape, got, ref)          # asserts TOL["bf16"] = 2e-2 for every tensor
    _report(shape.name, errs)
    plain = shape.with_(name="tp_share_175b_bf16_plain", fwd_fp16=False)
    got_plain = gpu_run(plain, params, xs, dys)
    errs_plain = compare(plain, got_plain, ref, tol=1.0)
    _report(plain.name, errs_plain)
    assert max(errs_plain.values()) > 1.5 * max(errs.values())


def test_workload4_full_size_decoupled():
    """The decoupled workload at full size in the launch configuration the benchmark
    times: 8 micro-batches, all forwards on one stream, then on another stream all backward
    data phases and one weight phase over the 8 micro-batches; 8 stash slots, one gradient
    buffer, PREPARED weight images.  The oracle cannot run all 8 micro-batches in test time, so:
      * against a second decoupled run on RAW weights with the weight gradients inside every
        backward call: y, dx of every micro-batch and every bias / LayerNorm gradient must
        agree bit for bit (same kernels, different operand layout), the weight matrices'
        gradients to 1e-5 of their maximum (the one-launch weight phase sums the 32768 tokens
        of all micro-batches in one fp32 accumulation instead of eight of 4096 added in
        fp32: both orders carry rounding of about sqrt(32768) * 2^-24 = 1e-5 of the sum's
        scale, three orders of magnitude under the bf16 bar);
      * y and dx of every micro-batch equal coupled single-micro-batch runs bit for bit;
      * the unsplit run's 8-micro-batch gradients equal, bit for bit, the fp32 sum (in call
        order) of the 8 single-micro-batch gradient buffers -- accumulation is `+=` into
        fp32, so this holds exactly and pins the accumulation semantics;
      * micro-batches 0 and 7 (first and last stash slot) are checked tensor by tensor
        against the oracle: y, dx, and the parameter gradients of their single runs."""
    shape = W[3]
    n = shape.n_microbatches
    print(f"[case] full {shape}", flush=True)
    params = synth.make_params(shape, 0)
    xs = [synth.make_x(shape, 0, m) for m in range(n)]
    dys = [synth.make_dy(shape, 0, m) for m in range(n)]
    bufs = B.StageBuffers(shape, n_stash=n)
    bufs.load_params(params)
    bufs.prepare()
    ys, dxs, g_split = gpu_run(shape, params, xs, dys, decoupled=True, bufs=bufs, split_wgrad=True)
    print("[step] decoupled 8 micro-batches, prepared weights, one weight phase: done", flush=True)
    bufs.unprepare()
    ys_raw, dxs_raw, g_all = gpu_run(shape, params, xs, dys, decoupled=True, bufs=bufs)
    for m in range(n):
        assert np.array_equal(ys[m], ys_raw[m]) and np.array_equal(dxs[m], dxs_raw[m]), m
    for la, lb in zip(g_split, g_all):
        for k in la:
            if k.startswith("w_"):
                assert max_norm_err(la[k], lb[k]) < 1e-5, k
            else:
                assert np.array_equal(la[k], lb[k]), k
    print("[step] benchmark configuration == raw weights / per-micro-batch weight gradients", flush=True)
    del ys_raw, dxs_raw, g_split
    bufs.prepare()
    acc = None
    singles = {}
    for m in range(n):
        y1, dx1, g1 = gpu_run(shape, params, [xs[m]], [dys[m]], decoupled=False, bufs=bufs)
        assert np.array_equal(y1[0], ys[m]) and np.array_equal(dx1[0], dxs[m]), m
        flat = [{k: v.astype(np.float32) for k, v in layer.items()} for layer in g1]
        if m in (0, n - 1):
            singles[m] = g1
        if m == 0:
            acc = flat
        else:
            for la, lb in zip(acc, flat):
                for k in la:
                    la[k] = la[k] + lb[k]          # fp32 adds in call order
    for la, lb in zip(acc, g_all):
        for k in la:
            assert np.array_equal(la[k].astype(np.float64), lb[k]), k
    print("[step] accumulation property holds; running the oracle on micro-batches 0 and 7", flush=True)
    del bufs, acc, g_all
    torch.cuda.empty_cache()
    for m in (0, n - 1):
        ref = oracle_run(shape, params, [xs[m]], [dys[m]])
        _report(f"{shape.name} micro-batch {m}", compare(shape, ([ys[m]], [dxs[m]], singles[m]), ref))


def test_boundary_contracts_dx_may_alias_dy_and_backward_keeps_the_stash():
    """Two promises of the header: dx may alias dy (the backward phase reads dy before the
    last kernel writes dx), and the backward phase does not modify the stash (running it
    twice on one stash gives the same bits)."""
    shape = W[1].with_(name="bf16_contracts", n_layers=2, hidden=512, n_heads=4, head_dim=128, ffn=1024,
                       seq=256, batch=2, bias_std=0.02, ln_jitter=0.1)
    print(f"[case] contracts {shape}", flush=True)
    params, xs, dys = _inputs(shape)
    bufs = B.StageBuffers(shape)
    bufs.load_params(params)
    p = bufs.params()
    x, dy = B.to_device(xs[0], shape.dtype), B.to_device(dys[0], shape.dtype)
    y, dx1, dx2 = bufs.act(), bufs.act(), bufs.act()
    B.gpt_stage_fwd(p, x, bufs.stash[0], y)
    stash_before = bufs.stash[0].clone()
    bufs.dparams.zero_()
    B.gpt_stage_bwd(p, bufs.stash[0], dy, dx1, bufs.dparams)
    g1 = bufs.dparams.clone()
    assert torch.equal(bufs.stash[0], stash_before)
    bufs.dparams.zero_()
    B.gpt_stage_bwd(p, bufs.stash[0], dy, dx2, bufs.dparams)
    assert torch.equal(dx1, dx2) and torch.equal(g1, bufs.dparams)
    alias = dy.clone()
    bufs.dparams.zero_()
    B.gpt_stage_bwd(p, bufs.stash[0], alias, alias, bufs.dparams)      # dx written over dy
    torch.cuda.synchronize()
    assert torch.equal(alias, dx1) and torch.equal(g1, bufs.dparams)


@pytest.mark.parametrize("dtype,hidden,ffn,seq,batch,layers", [("fp32", 128, 512, 3, 1, 1), ("fp32", 136, 200, 37, 7, 2),
                                                               ("bf16", 320, 832, 192, 2, 2), ("bf16", 1024, 1024, 64, 5, 1),
                                                               ("bf16", 1088, 1088, 320, 1, 1), ("bf16", 2048, 2048, 64, 1, 2)])
def test_bias_gradients_beside_the_layernorm(dtype, hidden, ffn, seq, batch, layers):
    """The column sums of a layer in the launch of its first LayerNorm's backward: each form of that kernel, one and
    several matrices, numbers of slices even and odd.  The same bits as from a launch of their own, which they have
    under a tracer and where a single layer's dx replaces dy."""
    shape = W[1].with_(name="bias_beside_ln", dtype=dtype, n_layers=layers, hidden=hidden, n_heads=2, head_dim=64, ffn=ffn,
                       seq=seq, batch=batch, bias_std=0.02, ln_jitter=0.1)
    print(f"[case] bias gradients beside the LayerNorm {shape}", flush=True)
    params, xs, dys = _inputs(shape)
    bufs = B.StageBuffers(shape)
    bufs.load_params(params)
    x, dy = B.to_device(xs[0], dtype), B.to_device(dys[0], dtype)
    y, dx = bufs.act(), bufs.act()
    B.gpt_stage_fwd(bufs.params(), x, bufs.stash[0], y)
    bufs.dparams.zero_()
    B.gpt_stage_bwd(bufs.params(), bufs.stash[0], dy, dx, bufs.dparams)
    together = bufs.dparams.clone()
    for traced in (False, True):
        bufs.trace = B.gpt_stage_trace_create(64) if traced else None
        over = dy.clone()
        bufs.dparams.zero_()
        B.gpt_stage_bwd(bufs.params(), bufs.stash[0], over, over, bufs.dparams)
        torch.cuda.synchronize()
        if traced:
            B.gpt_stage_trace_destroy(bufs.trace)
        assert torch.equal(over, dx) and torch.equal(bufs.dparams, together), traced


# ------------------------------------------------------- single operations ----
@pytest.mark.parametrize("dtype,layers,hidden,heads,ffn,seq,batch", [("fp32", 1, 128, 4, 512, 33, 2), ("fp32", 2, 136, 2, 200, 37, 3),
                                                                    ("bf16", 1, 320, 5, 832, 64, 1), ("bf16", 2, 192, 3, 2112, 96, 2),
                                                                    ("bf16", 3, 1024, 16, 4096, 320, 1), ("bf16", 2, 64, 1, 128, 64, 1),
                                                                    ("bf16", 1, 4096, 64, 4096, 1024, 16)])
@pytest.mark.parametrize("in_place", [False, True])
def test_partial_sums_beside_the_weight_gradients(dtype, layers, hidden, heads, ffn, seq, batch, in_place):
    """A layer's partial column sums are added up in the launch of its weight gradients, in one of their own under a tracer,
    where a single layer's dx lies on dy and where the gradients are a launch each (the last shape: whole rounds of tiles,
    16384 tokens): every output bit for bit the same either way, on widths that the matrix cores take in
    different tiles and on some that they do not take."""
    print(f"[case] sums beside wgrads {dtype} L={layers} H={hidden} F={ffn} T={seq * batch} {in_place}", flush=True)
    shape = synth.WORKLOADS[0].with_(name="sums_beside_wgrads", dtype=dtype, n_layers=layers, hidden=hidden, n_heads=heads,
                                     head_dim=64 if dtype == "bf16" else 32, ffn=ffn, seq=seq, batch=batch, bias_std=0.02, ln_jitter=0.1)
    bufs = B.StageBuffers(shape)
    bufs.load_params(synth.make_params(shape, 3))
    x, dy = B.to_device(synth.make_x(shape, 3), dtype), B.to_device(synth.make_dy(shape, 3), dtype)
    got = []
    for tracer in (None, B.gpt_stage_trace_create(4096)):
        bufs.trace = tracer
        bufs.dparams.fill_(0.125)
        y, g = bufs.act(), dy.clone()
        dx = g if in_place else bufs.act()
        B.gpt_stage_fwd(bufs.params(), x, bufs.stash[0], y)
        B.gpt_stage_bwd(bufs.params(), bufs.stash[0], g, dx, bufs.dparams)
        torch.cuda.synchronize()
        got.append((y, dx.clone(), bufs.dparams.clone()))
    bufs.trace = None
    B.gpt_stage_trace_destroy(tracer)
    for a, b in zip(*got):
        assert torch.equal(a, b)


@pytest.mark.parametrize("dtype,T,H,x_f32", [("fp32", 37, 128, False), ("fp32", 5, 4104, False),
                                             ("bf16", 130, 1024, False), ("bf16", 64, 12288, True),
                                             ("bf16", 3, 8, False), ("fp32", 600, 16384, False),
                                             ("bf16", 130, 1024, True), ("bf16", 7, 16384, True)])
def test_op_layernorm(dtype, T, H, x_f32):
    """x_f32: x is fp32 while gamma/beta/out/gradients are bf16 (the residual stream
    inside a bf16 stage)."""
    print(f"[case] layernorm {dtype} T={T} H={H} x_f32={x_f32}", flush=True)
    dt = B.GPTS_BF16 if dtype == "bf16" else B.GPTS_FP32
    x = synth.to_storage(synth.make_aux(0, 1, (T, H)) * 2 + 0.5, "fp32" if x_f32 else dtype)
    gam = synth.to_storage(1 + synth.make_aux(0, 2, (H,), 0.2), dtype)
    bet = synth.to_storage(synth.make_aux(0, 3, (H,), 0.2), dtype)
    dout = synth.to_storage(synth.make_aux(0, 4, (T, H)), dtype)
    dres = synth.to_storage(synth.make_aux(0, 5, (T, H)), dtype)
    dx_ = B.to_device(x, "fp32" if x_f32 else dtype)
    dg_, db_ = B.to_device(gam, dtype), B.to_device(bet, dtype)
    out = torch.empty_like(dg_.new_empty((T, H)))
    mean = torch.empty(T, dtype=torch.float32, device="cuda")
    rstd = torch.empty_like(mean)
    B.gpt_stage_op_layernorm_fwd(dt, T, H, 1e-5, dx_, dg_, db_, out, mean, rstd, x_f32=x_f32)
    ref_out, xhat, r = orc.layernorm_fwd(x, gam, bet, 1e-5)
    tol = TOL[dtype]
    assert max_norm_err(B.to_host(out), ref_out) <= tol
    assert max_norm_err(B.to_host(rstd), r[:, 0]) <= 1e-5
    assert max_norm_err(B.to_host(mean), x.astype(np.float64).mean(-1)) <= 1e-5
    part = torch.empty(B.gpt_stage_op_layernorm_bwd_scratch_bytes(T, H), dtype=torch.uint8, device="cuda")
    dgam = torch.full((H,), 1.0, dtype=torch.float32, device="cuda")     # pre-filled: += semantics
    dbet = torch.full((H,), -2.0, dtype=torch.float32, device="cuda")
    dxo = torch.empty_like(out)
    B.gpt_stage_op_layernorm_bwd(dt, T, H, B.to_device(dout, dtype), dx_, mean, rstd, dg_,
                                 B.to_device(dres, dtype), dxo, dgam, dbet, part, x_f32=x_f32)
    rdx, rdg, rdb = orc.layernorm_bwd(dout, xhat, r, gam)
    assert max_norm_err(B.to_host(dxo), rdx + dres) <= tol
    assert max_norm_err(B.to_host(dgam), rdg + 1.0) <= max(tol * 0.1, 1e-5)
    assert max_norm_err(B.to_host(dbet), rdb - 2.0) <= max(tol * 0.1, 1e-5)
    # same call with the column sums of dx requested (the fused bias gradient): dx, dgamma and
    # dbeta bit-identical to the call without, the sums += into a pre-filled vector
    dgam2 = torch.full((H,), 1.0, dtype=torch.float32, device="cuda")
    dbet2 = torch.full((H,), -2.0, dtype=torch.float32, device="cuda")
    dxs = torch.full((H,), 0.5, dtype=torch.float32, device="cuda")
    dxo2 = torch.empty_like(out)
    B.gpt_stage_op_layernorm_bwd(dt, T, H, B.to_device(dout, dtype), dx_, mean, rstd, dg_,
                                 B.to_device(dres, dtype), dxo2, dgam2, dbet2, part, x_f32=x_f32, dxsum=dxs)
    assert torch.equal(dxo2, dxo) and torch.equal(dgam2, dgam) and torch.equal(dbet2, dbet)
    assert max_norm_err(B.to_host(dxs), (rdx + dres).sum(0) + 0.5) <= max(tol * 0.1, 1e-5)


@pytest.mark.parametrize("dtype,T,H,x_f32", [("bf16", 5, 504, True), ("bf16", 2061, 512, True), ("fp32", 9, 520, False),
                                             ("bf16", 4100, 1024, True), ("fp32", 33, 1032, False), ("bf16", 515, 2048, True),
                                             ("bf16", 5, 2056, False), ("fp32", 513, 4096, False),
                                             ("fp32", 4100, 1160, False), ("fp32", 4097, 2048, False), ("bf16", 16390, 2048, True),
                                             ("bf16", 520, 12296, True)])
def test_op_layernorm_row_shapes(dtype, T, H, x_f32):
    """LayerNorm at the edges of its row shapes: a wave per row up to 1024 (backward) and 2048 (forward)
    columns, four waves up to 2048, a workgroup beyond and for many long rows; row counts that leave the last
    workgroup short."""
    test_op_layernorm(dtype, T, H, x_f32)


GEMM_SHAPES = [(64, 64, 64), (200, 136, 72), (256, 256, 256), (320, 448, 192), (512, 1024, 320),
               (1024, 768, 2048),
               (3904, 3392, 192),   # large enough for the 256x256 tiles, ragged last tile in M and N
               (3904, 3392, 384)]   # same with K a multiple of 128: the 16x16x32 kernels (NT and TN)


@pytest.mark.parametrize("dtype", ["fp32", "bf16"])
@pytest.mark.parametrize("M,N,K", GEMM_SHAPES)
def test_op_gemm_forms(dtype, M, N, K):
    print(f"[case] gemm {dtype} M={M} N={N} K={K}", flush=True)
    dt = B.GPTS_BF16 if dtype == "bf16" else B.GPTS_FP32
    tol = TOL[dtype]
    st = lambda tag, shp, std=1.0: synth.to_storage(synth.make_aux(1, tag, shp, std), dtype)
    dev = lambda a: B.to_device(a, dtype)
    # form 0: C = A B^T + bias (+ residual) ; gelu output
    A, Bm, bias, res = st(1, (M, K)), st(2, (N, K), 0.05), st(3, (N,), 0.5), st(4, (M, N))
    Cd = torch.empty((M, N), dtype=dev(A).dtype, device="cuda")
    B.gpt_stage_op_gemm(dt, 0, M, N, K, dev(A), dev(Bm), Cd, bias=dev(bias), residual=dev(res))
    ref = A.astype(np.float64) @ Bm.astype(np.float64).T + bias + res
    assert max_norm_err(B.to_host(Cd), ref) <= tol
    if dtype == "bf16":   # epilogues that extend the fp32 residual stream of a bf16 stage
        res32 = synth.make_aux(1, 8, (M, N))
        r32 = torch.from_numpy(res32).cuda()
        ref32 = A.astype(np.float64) @ Bm.astype(np.float64).T + bias + res32
        C32 = torch.empty((M, N), dtype=torch.float32, device="cuda")
        B.gpt_stage_op_gemm(dt, 0, M, N, K, dev(A), dev(Bm), C32, bias=dev(bias), residual=r32, f32_flags=3)
        assert max_norm_err(B.to_host(C32), ref32) <= 1e-3
        B.gpt_stage_op_gemm(dt, 0, M, N, K, dev(A), dev(Bm), Cd, bias=dev(bias), residual=r32, f32_flags=1)
        assert max_norm_err(B.to_host(Cd), ref32) <= tol
    for kind, variant in ((B.GPTS_GELU_TANH, "tanh"), (B.GPTS_GELU_ERF, "erf")):
        C2 = torch.empty_like(Cd)
        B.gpt_stage_op_gemm(dt, 0, M, N, K, dev(A), dev(Bm), Cd, bias=dev(bias), C2=C2, gelu_kind=kind)
        u = A.astype(np.float64) @ Bm.astype(np.float64).T + bias
        assert max_norm_err(B.to_host(Cd), u) <= tol
        assert max_norm_err(B.to_host(C2), orc.gelu(u, variant)) <= tol
    # form 1: C = A B (B is [K, N]) ; with the gelu' factor
    Bn, U = st(5, (K, N), 0.05), st(6, (M, N))
    B.gpt_stage_op_gemm(dt, 1, M, N, K, dev(A), dev(Bn), Cd)
    ref = A.astype(np.float64) @ Bn.astype(np.float64)
    assert max_norm_err(B.to_host(Cd), ref) <= tol
    B.gpt_stage_op_gemm(dt, 1, M, N, K, dev(A), dev(Bn), Cd, dgelu_u=dev(U))
    assert max_norm_err(B.to_host(Cd), ref * orc.gelu_grad(U, "tanh")) <= tol
    # form 2: Cf32 += A^T B, A is [K, M]
    At = st(7, (K, M))
    Cf = torch.full((M, N), 0.25, dtype=torch.float32, device="cuda")
    B.gpt_stage_op_gemm(dt, 2, M, N, K, dev(At), dev(Bn), Cf)
    ref = At.astype(np.float64).T @ Bn.astype(np.float64) + 0.25
    assert max_norm_err(B.to_host(Cf), ref) <= (1e-5 if dtype == "fp32" else 1e-4)


@pytest.mark.parametrize("M,N,K", [(1, 8, 4), (33, 36, 28), (31, 64, 124), (65, 100, 128), (32, 32, 132), (100, 516, 252),
                                   (64, 28, 260), (129, 260, 512), (999, 512, 516), (999, 1280, 260), (1030, 1540, 36),
                                   (1500, 2052, 100), (1500, 2052, 164), (1500, 2052, 292), (1500, 2052, 163)])
def test_op_gemm_fp32_slices(M, N, K):
    """Both fp32 tiles with ragged edges, and contractions that end at, just before and just behind a slice of 32, 64
    or 128 k, of one slice and of more than the slices ahead: the narrow tile up to 1280 columns, the 64 x 64 tile with two and
    four slices of 32, then six and ten, the last one short (163: the weight gradient's; the other two forms take whole
    fours of k, and other products the plain kernel).  What lies behind the operands is NaN.  A sum of K fp32
    products in any order is off by at most K eps of the sum of magnitudes."""
    print(f"[case] gemm fp32 slices M={M} N={N} K={K}", flush=True)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(M + N + K)

    def rnd(r, c):
        t = torch.full((r * c + 4096,), float("nan"), device="cuda")
        t[:r * c].normal_(generator=gen)
        return t[:r * c].view(r, c)

    for form in (0, 1, 2):
        m = (M + 3) // 4 * 4 if form == 2 else M
        A, Bm = (rnd(K, m) if form == 2 else rnd(m, K)), (rnd(N, K) if form == 0 else rnd(K, N))
        out = torch.full((m + 1, N), 0.25, device="cuda")
        B.gpt_stage_op_gemm(B.GPTS_FP32, form, m, N, K, A, Bm, out[:m])
        a, b = (A.double().t() if form == 2 else A.double()), (Bm.double().t() if form == 0 else Bm.double())
        ref = a @ b + (0.25 if form == 2 else 0.0)
        bound = (K + 1) * 2.0 ** -24 * (a.abs() @ b.abs() + 0.25)
        assert ((out[:m].double() - ref).abs() <= bound).all(), form
        assert (out[m] == 0.25).all(), form


def test_op_gemm_fp32_rows_of_more_than_32_bits_a_slice():
    """B's rows are so long that 128 of them, a slice of the narrow tile, are 4 GiB and 2 KiB: the product takes the
    other tile, whose slices are shorter.  Bound as above, on columns from the start, the middle and the end."""
    M, N, K = 4, (1 << 23) + 4, 132
    print(f"[case] gemm fp32 long rows M={M} N={N} K={K}", flush=True)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(4)
    A, Bm = (torch.empty(r, c, device="cuda").normal_(generator=gen) for r, c in ((M, K), (K, N)))
    out = torch.full((M, N), 7.0, device="cuda")
    B.gpt_stage_op_gemm(B.GPTS_FP32, 1, M, N, K, A, Bm, out)
    for c0 in (0, N // 2, N - 4096):
        a, b = A.double(), Bm[:, c0:c0 + 4096].double()
        assert ((out[:, c0:c0 + 4096].double() - a @ b).abs() <= (K + 1) * 2.0 ** -24 * (a.abs() @ b.abs())).all(), c0


@pytest.mark.parametrize("M,N,K", [(72, 1000, 64), (264, 3000, 128), (520, 2056, 192), (1000, 4104, 128), (2040, 4104, 128),
                                   (2040, 5112, 192), (2040, 6136, 64), (4088, 4088, 320), (264, 1000, 1024),
                                   (1000, 2056, 320), (8200, 4104, 64), (1000, 4104, 832), (2040, 4104, 832),
                                   (2040, 6136, 832), (1000, 2056, 832), (4088, 1160, 704), (8200, 4104, 768),
                                   (2568, 2056, 1088)])
def test_op_gemm_bf16_tiles(M, N, K):
    """Each tile of the bf16 products with ragged last tiles, one to sixteen slices, and the fp32 epilogues:
    weight gradients in 64x32, 64x64, 128x64, 192x192, 256x160, 256x256, 64x32 again with a long contraction,
    256x192, 128x128 on at most one a unit and on more, which share it, and 256x128 likewise; forward products and data gradients in the same tiles, except
    that up to 768 k the shapes of more than 256 tiles of 128x64 take 128x64 and 128x128 in two
    stages; then the tiles passed over for those, with 832 k, and both of the two-stage forms with eleven
    and twelve slices.  fp32 sums of K products of bf16 values: K eps of the sum of magnitudes."""
    print(f"[case] gemm tiles M={M} N={N} K={K}", flush=True)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(M + N + K)
    rnd = lambda *s: torch.empty(s, dtype=torch.bfloat16, device="cuda").normal_(generator=gen)
    A, Bt, At, U, bias = rnd(M, K), rnd(N, K), rnd(K, M), rnd(M, N), rnd(N)
    res = torch.empty(M, N, dtype=torch.float32, device="cuda").normal_(generator=gen)
    bound = 4 * K ** 0.5 * K * 2.0 ** -24 + 1e-6          # of fp32 outputs with |a b| of order 1
    ref = A.double() @ Bt.double().T
    out = torch.full((M, N), 7.0, dtype=torch.float32, device="cuda")
    B.gpt_stage_op_gemm(B.GPTS_BF16, 0, M, N, K, A, Bt, out, bias=bias, residual=res, f32_flags=3)
    assert (out.double() - (ref + bias.double() + res.double())).abs().max().item() <= bound + 2.0 ** -22 * K ** 0.5
    out = torch.full((M, N), 0.25, dtype=torch.float32, device="cuda")
    Bn = Bt.T.contiguous()
    B.gpt_stage_op_gemm(B.GPTS_BF16, 2, M, N, K, At, Bn, out)
    assert (out.double() - (At.double().T @ Bn.double() + 0.25)).abs().max().item() <= bound + 2.0 ** -22 * K ** 0.5
    # data gradient with the GeLU' factor: rounded once to bf16 (2^-9 of the value)
    out = torch.full((M, N), 7.0, dtype=torch.bfloat16, device="cuda")
    B.gpt_stage_op_gemm(B.GPTS_BF16, 1, M, N, K, A, Bn, out, dgelu_u=U)
    u = U.double().requires_grad_()
    torch.nn.functional.gelu(u, approximate="tanh").sum().backward()
    want = ref * u.grad
    assert ((out.double() - want).abs() <= want.abs() * 2.0 ** -8 + 2.0 ** -12 * K ** 0.5).all()


@pytest.mark.parametrize("gelu", ["tanh", "erf"])
@pytest.mark.parametrize("M,N,K", [(2040, 4104, 64), (2056, 4088, 128), (4088, 4096, 64), (4104, 4096, 64), (4088, 4112, 320),
                                   (8200, 2056, 832), (2568, 8200, 1088)])
def test_op_gemm_bf16_matrices_around_the_size_of_the_caches(M, N, K, gelu):
    """Accumulated fp32 matrices and pre-activations on both sides of 32 MB, from which on their accesses are
    non-temporal.  u and the gradient through GeLU' are rounded once to bf16 (2^-9 of the value), g = gelu(u as stored) likewise."""
    print(f"[case] once M={M} N={N} K={K} {gelu}", flush=True)
    kind = B.GPTS_GELU_TANH if gelu == "tanh" else B.GPTS_GELU_ERF
    gen = torch.Generator(device="cuda")
    gen.manual_seed(M + N + K)
    rnd = lambda *s: torch.empty(s, dtype=torch.bfloat16, device="cuda").normal_(generator=gen)
    A, Bt, U, bias = rnd(M, K), rnd(N, K), rnd(M, N), rnd(N)
    u, g = torch.full((M, N), 7.0, dtype=torch.bfloat16, device="cuda"), torch.full((M, N), 7.0, dtype=torch.bfloat16, device="cuda")
    B.gpt_stage_op_gemm(B.GPTS_BF16, 0, M, N, K, A, Bt, u, bias=bias, C2=g, gelu_kind=kind)
    ref = A.double() @ Bt.double().T
    slack = 2.0 ** -12 * K ** 0.5
    assert ((u.double() - ref - bias.double()).abs() <= (ref + bias.double()).abs() * 2.0 ** -8 + slack).all()
    want = torch.nn.functional.gelu(u.double(), approximate="tanh" if gelu == "tanh" else "none")
    assert ((g.double() - want).abs() <= want.abs() * 2.0 ** -8 + 1e-5).all()
    out = torch.full((M, N), 7.0, dtype=torch.bfloat16, device="cuda")
    Bn = Bt.T.contiguous()
    B.gpt_stage_op_gemm(B.GPTS_BF16, 1, M, N, K, A, Bn, out, dgelu_u=U, gelu_kind=kind)
    v = U.double().requires_grad_()
    torch.nn.functional.gelu(v, approximate="tanh" if gelu == "tanh" else "none").sum().backward()
    want = ref * v.grad
    assert ((out.double() - want).abs() <= want.abs() * 2.0 ** -8 + slack).all()
    At = A.T.contiguous()
    acc = torch.full((M, N), 0.25, dtype=torch.float32, device="cuda")
    B.gpt_stage_op_gemm(B.GPTS_BF16, 2, M, N, K, At, Bn, acc)
    B.gpt_stage_op_gemm(B.GPTS_BF16, 2, M, N, K, At, Bn, acc)      # reads what the first call wrote
    bound = 4 * K ** 0.5 * K * 2.0 ** -24 + 1e-6
    assert (acc.double() - (2 * ref + 0.25)).abs().max().item() <= 2 * bound + 2.0 ** -21 * K ** 0.5


@pytest.mark.parametrize("M,N,K", [(520, 1032, 65600), (264, 3000, 32768)])
def test_op_gemm_bf16_wgrad_large_operands(M, N, K):
    """Weight gradients whose operands exceed the cache (above 200 MB tiles are chosen by another rate), ragged in
    both widths.  fp32 sums of K/32 matrix steps: errors of sqrt(K/32) roundings of 2^-24 in the 2-norm, four
    times that allowed."""
    print(f"[case] wgrad of large operands M={M} N={N} K={K}", flush=True)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(K)
    A, Bn = (torch.empty(K, w, dtype=torch.bfloat16, device="cuda").normal_(generator=gen) for w in (M, N))
    out = torch.full((M, N), 0.25, dtype=torch.float32, device="cuda")
    B.gpt_stage_op_gemm(B.GPTS_BF16, 2, M, N, K, A, Bn, out)
    want = A.double().t().contiguous() @ Bn.double() + 0.25
    assert ((out.double() - want).norm() / want.norm()).item() <= 4 * (K / 32) ** 0.5 * 2.0 ** -24


@pytest.mark.parametrize("M,N,K", [(1, 4, 4), (33, 36, 60), (32, 32, 64), (31, 100, 68), (65, 60, 132), (4, 4, 1),
                                   (36, 64, 999), (1216, 1032, 40), (1100, 1284, 36), (8, 6, 8), (10, 12, 7)])
def test_op_gemm_fp32_edges(M, N, K):
    """The fp32 matrix-core products at the edges of their two tile sizes (32 and 64), of the slices
    (64 and 32) and of the rule between them, and the widths that are left to the plain kernel.
    Every element within (K + 4) roundings of its sum of magnitudes."""
    print(f"[case] gemm fp32 edges M={M} N={N} K={K}", flush=True)
    dt, dev = B.GPTS_FP32, lambda a: B.to_device(a, "fp32")
    eps = (K + 4) * 2.0 ** -23
    mk = lambda tag, shp: synth.to_storage(synth.make_aux(11, tag, shp), "fp32")
    A, Bm, bias, res, At, Bn = mk(1, (M, K)), mk(2, (N, K)), mk(3, (N,)), mk(4, (M, N)), mk(5, (K, M)), mk(6, (K, N))
    f64 = lambda a: a.astype(np.float64)
    Cd = torch.empty((M, N), dtype=torch.float32, device="cuda")

    def check(got, ref, mag):
        assert (np.abs(B.to_host(got) - ref) <= eps * mag).all()

    B.gpt_stage_op_gemm(dt, 0, M, N, K, dev(A), dev(Bm), Cd, bias=dev(bias), residual=dev(res))
    check(Cd, f64(A) @ f64(Bm).T + bias + res, np.abs(f64(A)) @ np.abs(f64(Bm)).T + np.abs(bias) + np.abs(res))
    B.gpt_stage_op_gemm(dt, 1, M, N, K, dev(A), dev(Bn), Cd)
    check(Cd, f64(A) @ f64(Bn), np.abs(f64(A)) @ np.abs(f64(Bn)))
    Cf = dev(res)
    B.gpt_stage_op_gemm(dt, 2, M, N, K, dev(At), dev(Bn), Cf)
    check(Cf, f64(At).T @ f64(Bn) + res, np.abs(f64(At)).T @ np.abs(f64(Bn)) + np.abs(res))


@pytest.mark.parametrize("dtype,M,N", [("fp32", 100, 136), ("bf16", 4096, 1024), ("bf16", 7, 8), ("bf16", 1000, 4608)])
def test_op_colsum(dtype, M, N):
    print(f"[case] colsum {dtype} M={M} N={N}", flush=True)
    dt = B.GPTS_BF16 if dtype == "bf16" else B.GPTS_FP32
    A = synth.to_storage(synth.make_aux(2, 1, (M, N)), dtype)
    out = torch.full((N,), 3.0, dtype=torch.float32, device="cuda")
    part = torch.empty(B.gpt_stage_op_colsum_scratch_bytes(M, N), dtype=torch.uint8, device="cuda")
    B.gpt_stage_op_colsum(dt, M, N, B.to_device(A, dtype), out, part)
    assert max_norm_err(B.to_host(out), A.astype(np.float64).sum(0) + 3.0) <= 1e-5


@pytest.mark.parametrize("dtype,Bn,S,a,d", [("fp32", 2, 64, 4, 32), ("fp32", 1, 97, 2, 64), ("bf16", 2, 256, 3, 64),
                                            ("bf16", 1, 384, 2, 128), ("bf16", 1, 1, 2, 64), ("fp32", 1, 130, 1, 128),
                                            ("bf16", 2, 1000, 2, 128), ("bf16", 1, 777, 3, 64), ("bf16", 1, 2048, 1, 128),
                                            ("bf16", 3, 50, 2, 32), ("bf16", 2, 700, 3, 32)])
def test_op_attention(dtype, Bn, S, a, d):
    print(f"[case] attention {dtype} B={Bn} S={S} a={a} d={d}", flush=True)
    dt = B.GPTS_BF16 if dtype == "bf16" else B.GPTS_FP32
    tol = TOL[dtype]
    P = a * d
    qkv = synth.to_storage(synth.make_aux(3, 1, (Bn, S, 3 * P)), dtype)
    dout = synth.to_storage(synth.make_aux(3, 2, (Bn, S, P)), dtype)
    qd = B.to_device(qkv, dtype)
    out = torch.empty((Bn, S, P), dtype=qd.dtype, device="cuda")
    lse = torch.empty((Bn, a, S), dtype=torch.float32, device="cuda")
    scratch = [torch.empty(max(B.gpt_stage_op_attention_scratch_bytes(dt, Bn, S, a, d, ph), 256),
                           dtype=torch.uint8, device="cuda") for ph in (0, 1)]
    B.gpt_stage_op_attention_fwd(dt, Bn, S, a, d, qd, out, lse, scratch[0])
    ref = orc.attention_fwd(qkv, a, d)
    assert max_norm_err(B.to_host(out), ref) <= tol
    # lse against its definition: log sum_{j<=i} exp(q_i.k_j/sqrt(d))
    q64 = qkv.astype(np.float64)
    ref_lse = np.empty((Bn, a, S))
    for b in range(Bn):
        for n in range(a):
            s = q64[b, :, n * d:(n + 1) * d] @ q64[b, :, P + n * d:P + (n + 1) * d].T / np.sqrt(d)
            s = np.where(np.tril(np.ones((S, S), bool)), s, -np.inf)
            m = s.max(1)
            ref_lse[b, n] = m + np.log(np.exp(s - m[:, None]).sum(1))
    assert np.abs(B.to_host(lse) - ref_lse).max() <= 1e-4 * max(1.0, np.abs(ref_lse).max())
    dqkv = torch.empty_like(qd)
    B.gpt_stage_op_attention_bwd(dt, Bn, S, a, d, qd, out, lse, B.to_device(dout, dtype), dqkv, scratch[1])
    rd = orc.attention_bwd(qkv, dout, a, d)
    got = B.to_host(dqkv)
    for i, nm in enumerate("qkv"):
        assert max_norm_err(got[..., i * P:(i + 1) * P], rd[..., i * P:(i + 1) * P]) <= tol, f"d{nm}"


def _attention_op(dt, Bn, S, a, d, qkv, dout):
    """(out, lse, dqkv) of the attention operators on device tensors."""
    out = torch.empty((Bn, S, a * d), dtype=qkv.dtype, device="cuda")
    lse = torch.empty((Bn, a, S), dtype=torch.float32, device="cuda")
    dqkv = torch.empty_like(qkv)
    scratch = [torch.empty(max(B.gpt_stage_op_attention_scratch_bytes(dt, Bn, S, a, d, ph), 256),
                           dtype=torch.uint8, device="cuda") for ph in (0, 1)]
    B.gpt_stage_op_attention_fwd(dt, Bn, S, a, d, qkv, out, lse, scratch[0])
    B.gpt_stage_op_attention_bwd(dt, Bn, S, a, d, qkv, out, lse, dout, dqkv, scratch[1])
    return out, lse, dqkv


@pytest.mark.parametrize("Bn,S,a,d", [(1, 1, 1, 32), (1, 31, 2, 64), (2, 33, 3, 128), (1, 65, 3, 32), (1, 97, 2, 64), (1, 129, 2, 128),
                                      (3, 320, 14, 64), (1, 1000, 9, 128), (1, 257, 130, 32), (1, 260, 150, 64), (1, 130, 300, 128),
                                      (1, 300, 260, 32), (1, 200, 200, 64), (1, 161, 150, 64), (1, 193, 120, 128), (1, 130, 230, 128),
                                      (1, 520, 60, 128), (1, 520, 84, 128), (1, 520, 83, 128)])
def test_op_attention_bf16_splits(Bn, S, a, d):
    """The arrangements of the bf16 attention kernels at the edges of their blocks (32, 64, 128, 256 rows): waves
    per 32 rows in forward and backward, in order: two and one, twice one and one, five times two and two, two and
    one, four times one and one, twice two and one, one and one, two and one, twice one and one.
    Against fp64 on the same inputs; probabilities, dS and the outputs are rounded to bf16
    (2^-9 each), so 2-norm errors stay within 2^-7 and single values within 2^-4 of the largest."""
    print(f"[case] attention splits B={Bn} S={S} a={a} d={d}", flush=True)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(S * a + d)
    qkv = torch.empty(Bn, S, 3 * a * d, dtype=torch.bfloat16, device="cuda").normal_(generator=gen)
    dout = torch.empty(Bn, S, a * d, dtype=torch.bfloat16, device="cuda").normal_(generator=gen)
    out, dqkv = torch.full_like(dout, 7.0), torch.full_like(qkv, 7.0)
    lse = torch.full((Bn, a, S), 7.0, dtype=torch.float32, device="cuda")
    scratch = [torch.empty(max(B.gpt_stage_op_attention_scratch_bytes(B.GPTS_BF16, Bn, S, a, d, ph), 256),
                           dtype=torch.uint8, device="cuda") for ph in (0, 1)]
    B.gpt_stage_op_attention_fwd(B.GPTS_BF16, Bn, S, a, d, qkv, out, lse, scratch[0])
    B.gpt_stage_op_attention_bwd(B.GPTS_BF16, Bn, S, a, d, qkv, out, lse, dout, dqkv, scratch[1])
    masked = torch.ones(S, S, dtype=torch.bool, device="cuda").triu(1)
    for b in range(Bn):
        x = qkv[b].double().requires_grad_()
        q, k, v = (t.reshape(S, a, d).transpose(0, 1).contiguous() for t in x.split(a * d, dim=1))
        s = torch.stack([q[n] @ k[n].t() for n in range(a)]) / d ** 0.5
        s = s.masked_fill(masked, float("-inf"))
        o = torch.stack([torch.softmax(s[n], -1) @ v[n] for n in range(a)]).transpose(0, 1).reshape(S, a * d)
        o.backward(dout[b].double())
        assert (lse[b].double() - torch.logsumexp(s.detach(), -1)).abs().max().item() < 1e-5
        for got, want in ((out[b].double(), o.detach()), (dqkv[b].double(), x.grad)):
            assert ((got - want).norm() / want.norm()).item() < 2 ** -7
            assert (got - want).abs().max().item() < 2 ** -4 * want.abs().max().item()


@pytest.mark.parametrize("Bn,S,a,d", [(1, 130, 90, 128), (1, 100, 150, 64), (2, 70, 200, 32), (1, 130, 600, 128), (2, 70, 430, 64),
                                      (1, 65, 900, 32), (1, 449, 220, 128)])
def test_op_attention_bf16_backward_forms(Bn, S, a, d):
    """One wave per 32 rows in backward: 128 rows and one launch (the first three), 128 rows and a launch for each
    side (the next three), 256 rows.  Reference and tolerances as in test_op_attention_bf16_splits."""
    test_op_attention_bf16_splits(Bn, S, a, d)


def test_op_attention_bf16_as_many_sequences_as_a_launch_takes():
    """65536 sequences of one token: its probability is 1, so out is v, dV is dO, and dS, which is 0, is what two orders of a sum of
    32 products of about 1 differ by, at most 32 eps times them."""
    Bn, d = 65536, 32
    print(f"[case] attention sequences={Bn}", flush=True)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(9)
    qkv = torch.empty(Bn, 1, 3 * d, dtype=torch.bfloat16, device="cuda").normal_(generator=gen)
    dout = torch.empty(Bn, 1, d, dtype=torch.bfloat16, device="cuda").normal_(generator=gen)
    out, lse, dqkv = _attention_op(B.GPTS_BF16, Bn, 1, 1, d, qkv, dout)
    q, k, v = qkv.float().split(d, dim=2)
    assert torch.equal(out.float(), v) and torch.equal(dqkv[..., 2 * d:], dout)
    assert ((q * k).sum(2).view(-1) / d ** 0.5 - lse.view(-1)).abs().max().item() < 1e-5
    ds = 32 * 2.0 ** -23 * (dout.float() * v).abs().sum(2, keepdim=True) + 2.0 ** -126
    assert (dqkv[..., :d].float().abs() <= ds * k.abs()).all() and (dqkv[..., d:2 * d].float().abs() <= ds * q.abs()).all()


@pytest.mark.parametrize("S,few,many,d", [(130, 56, 60, 32), (130, 56, 60, 64), (130, 56, 60, 128), (449, 21, 22, 128)])
def test_op_attention_bf16_forms_with_one_wave_agree_bit_for_bit(S, few, many, d):
    """A sequence's results do not depend on how many others there are, while one wave takes 32 rows: backward in one
    launch and in a launch for each side, 128 rows (the first three) and 256."""
    print(f"[case] attention forms agree S={S} sequences={few},{many} d={d}", flush=True)
    a = 10
    gen = torch.Generator(device="cuda")
    gen.manual_seed(S)
    qkv = torch.empty(many, S, 3 * a * d, dtype=torch.bfloat16, device="cuda").normal_(generator=gen)
    dout = torch.empty(many, S, a * d, dtype=torch.bfloat16, device="cuda").normal_(generator=gen)
    want = _attention_op(B.GPTS_BF16, few, S, a, d, qkv[:few], dout[:few])
    got = _attention_op(B.GPTS_BF16, many, S, a, d, qkv, dout)
    for name, x, y in zip(("out", "lse", "dqkv"), got, want):
        assert torch.equal(x[:few], y), name


_KEY_SIDE_FORMS = pytest.mark.parametrize("S,a", [(32, 2), (70, 2), (128, 300), (130, 1200)])   # 64 rows, 128, 128 in a launch for each side


def _attention_bwd_op(qkv, out, lse, dout):
    _, S, _, a, d = qkv.shape
    scratch = torch.empty(max(B.gpt_stage_op_attention_scratch_bytes(B.GPTS_BF16, 1, S, a, d, 1), 256), dtype=torch.uint8, device="cuda")
    dqkv = torch.full_like(qkv, 7.0)
    B.gpt_stage_op_attention_bwd(B.GPTS_BF16, 1, S, a, d, qkv, out, lse, dout, dqkv, scratch)
    return dqkv[0].float()


@_KEY_SIDE_FORMS
def test_op_attention_bf16_key_side_exponent_rounds_at_the_size_of_the_difference(S, a):
    """Logits of 2^20 for the last query and an lse 3/8 above them, both whole eighths: P = exp(-3/8) but for the roundings of the
    difference, of log2(e) and of the power, under 2^-20 together, so dV is 32 times bf16(P) (175.95/256, far from a tie).
    The other queries' P is 0 (lse 2^20 above their logits)."""
    print(f"[case] attention key side exponent S={S} a={a}", flush=True)
    qkv = torch.zeros(1, S, 3, a, 64, dtype=torch.bfloat16, device="cuda")
    out, dout = torch.zeros(2, 1, S, a, 64, dtype=torch.bfloat16, device="cuda")
    lse = torch.full((1, a, S), 2.0 ** 20, device="cuda")
    qkv[:, -1, 0, :, 0] = 2.0 ** 12
    qkv[:, :, 1, :, 0] = 2.0 ** 11
    dout[:, -1] = 32.0
    lse[:, :, -1] += 0.375
    dv = _attention_bwd_op(qkv, out, lse, dout)[:, 2]
    assert torch.equal(dv, torch.full_like(dv, 32.0 * 176 / 256))


@_KEY_SIDE_FORMS
def test_op_attention_bf16_key_side_takes_delta_from_the_whole_dp(S, a):
    """delta = -(2^24 + 2^16), halfway between two bf16 values, and dP = 4, one from every 16 columns: dP - delta is
    2^24 + 2^16 + 4 exactly and rounds up; a sum that began at -delta would stay halfway.  The last query's P is 1 (logits and lse
    0), the others' 0, and dK = dS q / sqrt(64)."""
    print(f"[case] attention key side delta S={S} a={a}", flush=True)
    qkv = torch.zeros(1, S, 3, a, 64, dtype=torch.bfloat16, device="cuda")
    out, dout = torch.zeros(2, 1, S, a, 64, dtype=torch.bfloat16, device="cuda")
    lse = torch.full((1, a, S), 2.0 ** 20, device="cuda")
    lse[:, :, -1] = 0.0
    qkv[:, -1, 0, :, 1] = 1.0                   # (K is 0: the logits stay 0)
    qkv[:, :, 2, :, ::16] = 2.0 ** -12
    dout[:, -1, :, ::16] = 2.0 ** 12
    out[:, -1, :, 0] = -(2.0 ** 12)
    out[:, -1, :, 16] = -(2.0 ** 4)
    dk = _attention_bwd_op(qkv, out, lse, dout)[:, 1, :, 1]
    assert torch.equal(dk, torch.full_like(dk, (2.0 ** 24 + 2.0 ** 17) / 8))


@pytest.mark.parametrize("S,few,many", [(1000, 100, 128), (1030, 64, 90), (1279, 60, 102), (1281, 60, 80),
                                        (1500, 60, 80), (2047, 50, 60), (2230, 45, 110), (5633, 18, 20)])
def test_op_attention_bf16_forward_in_eight_waves(S, few, many):
    """Many long sequences of head dimension 128 go in workgroups of eight waves, fewer in four: the same bits.  (The first four
    are on the four-wave side of the limits whatever their number, the others reach eight waves: one pair of rounds, two, and
    a last workgroup of one row.)  Keys 4 .. 7 of
    every eight have logits eight times as large, so that the maximum is in the other half of the wave from half of the
    keys; against 64 bits: out rounds to bf16 the sum of probabilities rounded to bf16."""
    print(f"[case] attention forward eight waves S={S} sequences={few},{many}", flush=True)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(S)
    qkv = torch.empty(many, S, 3 * 128, dtype=torch.bfloat16, device="cuda").normal_(generator=gen)
    big = torch.arange(S, device="cuda") % 8 >= 4
    qkv[:, big, 128:256] *= 8
    got = []
    for n in (many, few):
        out = torch.full((n, S, 128), 7.0, dtype=torch.bfloat16, device="cuda")
        lse = torch.full((n, 1, S), 7.0, device="cuda")
        scratch = torch.empty(256, dtype=torch.uint8, device="cuda")
        B.gpt_stage_op_attention_fwd(B.GPTS_BF16, n, S, 1, 128, qkv[:n].contiguous(), out, lse, scratch)
        got.append((out, lse))
    assert torch.equal(got[0][0][:few], got[1][0]) and torch.equal(got[0][1][:few], got[1][1])
    q, k, v = (t.double() for t in qkv[many - 1].split(128, dim=1))
    s = (q @ k.t() / 128 ** 0.5).masked_fill(torch.ones(S, S, dtype=torch.bool, device="cuda").triu(1), float("-inf"))
    p = torch.softmax(s, dim=-1)
    bound = 2.0 ** -8 * (p @ v.abs()) + 2.0 ** -8 * (p @ v).abs() + 1e-6
    assert ((got[0][0][many - 1].double() - p @ v).abs() <= bound).all()
    assert (got[0][1][many - 1, 0].double() - torch.logsumexp(s, dim=-1)).abs().max().item() <= 1e-4


def test_fp16_stage_with_the_attention_forward_in_eight_waves():
    """fp16 forward activations, 20 sequences of 1504 tokens in 4 heads of 128: 480 workgroups of 256 rows, the last with 224,
    take eight waves; 16 sequences take four (384 workgroups are not nearly a pair of rounds).  The same bits, and the last
    two sequences as the oracle has them."""
    shape = W[1].with_(name="fp16_eight_waves", n_layers=1, hidden=128, n_heads=4, head_dim=128, ffn=128, seq=1504, batch=20,
                       bias_std=0.02, ln_jitter=0.1, fwd_fp16=True)
    print(f"[case] stage {shape}", flush=True)
    params, xs, dys = _inputs(shape)
    got = []
    for n in (20, 16):
        y, dx, _ = gpu_run(shape.with_(batch=n), params, [xs[0][:n]], [dys[0][:n]])
        got.append((y[0], dx[0]))
    assert np.array_equal(got[0][0][:16], got[1][0])
    ref_y, ref_dx, _ = oracle_run(shape, params, [xs[0][18:]], [dys[0][18:]])
    for g, r in zip(got[0], (ref_y[0], ref_dx[0])):
        assert max_norm_err(g[18:], r) <= TOL["bf16"]


@pytest.mark.parametrize("S,a,d", [(70, 2, 128), (97, 1, 64), (65, 3, 32), (70, 500, 64)])
def test_op_attention_bf16_rows_past_the_end_count_as_zeros(S, a, d):
    """The last tile's rows past the sequence's end hold a copy of its last row: with an infinite value there
    (and in its output gradient) the last query's output is infinite and no NaN, and the last key's dV too."""
    print(f"[case] attention rows past the end S={S} a={a} d={d}", flush=True)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(S)
    qkv = torch.empty(1, S, 3, a, d, dtype=torch.bfloat16, device="cuda").normal_(generator=gen)
    dout = torch.empty(1, S, a, d, dtype=torch.bfloat16, device="cuda").normal_(generator=gen)
    finite = _attention_op(B.GPTS_BF16, 1, S, a, d, qkv, dout)
    qkv[:, -1, 2] = float("inf")
    out, lse, _ = _attention_op(B.GPTS_BF16, 1, S, a, d, qkv, dout)
    assert (out[0, -1] == float("inf")).all() and torch.equal(lse, finite[1])
    qkv[:, -1, 2] = 1.0
    dout[:, -1] = float("inf")
    dv = _attention_op(B.GPTS_BF16, 1, S, a, d, qkv, dout)[2].view(S, 3, a, d)[:, 2]
    assert (dv[-1] == float("inf")).all()


@pytest.mark.parametrize("Bn,S,a,d", [(1, 40, 2, 64), (1, 97, 2, 128), (2, 130, 1, 32), (1, 70, 300, 32), (1, 97, 3, 64)])
def test_op_attention_bf16_minus_infinite_logits(Bn, S, a, d):
    """Keys 32 to 63, the second wave's share of the first tile where two waves take a row block (all but the
    first), have logits of -inf for every query: they count as masked keys do, in the output and in lse.
    Tolerances as in test_op_attention_bf16_splits."""
    print(f"[case] attention minus infinity B={Bn} S={S} a={a} d={d}", flush=True)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(S * a + d)
    qkv = torch.empty(Bn, S, 3, a, d, dtype=torch.bfloat16, device="cuda").normal_(generator=gen)
    qkv[:, :, 0, :, 0] = -1.0
    qkv[:, 32:64, 1, :, 0] = float("inf")
    out = torch.full((Bn, S, a * d), 7.0, dtype=torch.bfloat16, device="cuda")
    lse = torch.full((Bn, a, S), 7.0, dtype=torch.float32, device="cuda")
    scratch = torch.empty(max(B.gpt_stage_op_attention_scratch_bytes(B.GPTS_BF16, Bn, S, a, d, 0), 256), dtype=torch.uint8, device="cuda")
    B.gpt_stage_op_attention_fwd(B.GPTS_BF16, Bn, S, a, d, qkv, out, lse, scratch)
    x = qkv.cpu().double()
    x[:, 32:64, 1, :, 0] = 0.0
    masked = torch.ones(S, S, dtype=torch.bool).triu(1)
    masked[:, 32:64] = True
    for b in range(Bn):
        q, k, v = (t.transpose(0, 1).contiguous() for t in x[b].unbind(1))
        s = (torch.stack([q[n] @ k[n].t() for n in range(a)]) / d ** 0.5).masked_fill(masked, float("-inf"))
        want = torch.stack([torch.softmax(s[n], -1) @ v[n] for n in range(a)]).transpose(0, 1).reshape(S, a * d)
        got = out[b].cpu().double()
        assert (lse[b].cpu().double() - torch.logsumexp(s, -1)).abs().max().item() < 1e-5
        assert ((got - want).norm() / want.norm()).item() < 2 ** -7
        assert (got - want).abs().max().item() < 2 ** -4 * want.abs().max().item()


@pytest.mark.parametrize("Bn,S,a,d", [(1, 1, 1, 32), (2, 15, 2, 64), (1, 16, 2, 128), (2, 17, 3, 32), (1, 63, 1, 128),
                                      (1, 65, 2, 64), (2, 130, 2, 32)])
def test_op_attention_fp32_edges(Bn, S, a, d):
    """The fp32 matrix-core attention at the edges of its 16-row blocks and of the four waves' turns
    (64 rows); a token that is not finite touches no row that cannot see it."""
    print(f"[case] attention fp32 edges B={Bn} S={S} a={a} d={d}", flush=True)
    P = a * d
    qkv = synth.to_storage(synth.make_aux(12, 1, (Bn, S, 3 * P)), "fp32")
    dout = synth.to_storage(synth.make_aux(12, 2, (Bn, S, P)), "fp32")
    qd, dd = B.to_device(qkv, "fp32"), B.to_device(dout, "fp32")
    out, lse, dqkv = _attention_op(B.GPTS_FP32, Bn, S, a, d, qd, dd)
    # sums of at most S products of O(1) terms in fp32, exponents of magnitude below 32: 32 * S * 2^-24
    tol = max(1e-5, 32 * S * 2.0 ** -24)
    assert max_norm_err(B.to_host(out), orc.attention_fwd(qkv, a, d)) <= tol
    assert max_norm_err(B.to_host(dqkv), orc.attention_bwd(qkv, dout, a, d)) <= tol
    if S == 1:
        return

    def same(got, want):   # the same sums in another order: within the tolerance above, NaN never
        assert max_norm_err(B.to_host(got), B.to_host(want)) <= tol

    bad_last, bad_dout = qd.clone(), dd.clone()   # the last token: nothing before it sees its key and value
    bad_last[:, -1] = float("nan")
    o2, l2, g2 = _attention_op(B.GPTS_FP32, Bn, S, a, d, bad_last, bad_dout)
    same(o2[:, :-1], out[:, :-1])
    same(l2[..., :-1], lse[..., :-1])
    same(g2[:, :-1, :P], dqkv[:, :-1, :P])
    bad_first, bad_dout = qd.clone(), dd.clone()   # the first query: it sees no later key
    bad_first[:, 0, :P] = float("inf")
    bad_dout[:, 0] = float("inf")
    o3, _, g3 = _attention_op(B.GPTS_FP32, Bn, S, a, d, bad_first, bad_dout)
    same(o3[:, 1:], out[:, 1:])
    same(g3[:, 1:, P:], dqkv[:, 1:, P:])


@pytest.mark.gpu
@pytest.mark.parametrize("dtype", ["fp32", "bf16"])
def test_recompute_variant_identical_results_smaller_stash(dtype):
    """Activation recomputation (sections 4.1 / 5.2): the backward phase rebuilds the
    LayerNorm and GeLU outputs instead of reading them from the stash.  Same bits, smaller
    stash; checked against the oracle too."""
    shape = synth.StageShape(name="rc", n_layers=2, hidden=256, n_heads=2, head_dim=64, ffn=512, seq=192,
                             batch=2, dtype=dtype, n_microbatches=2, bias_std=0.02, ln_jitter=0.1)
    print(f"[case] recompute {dtype}", flush=True)
    params = [{k: synth.to_storage(v, dtype) for k, v in synth.make_layer_params(shape, l, 0).items()}
              for l in range(shape.n_layers)]
    xs = [synth.to_storage(synth.make_x(shape, 0, m), dtype) for m in range(2)]
    dys = [synth.to_storage(synth.make_dy(shape, 0, m), dtype) for m in range(2)]
    full = gpu_run(shape, params, xs, dys, decoupled=True)
    rshape = shape.with_(recompute=True)
    rec = gpu_run(rshape, params, xs, dys, decoupled=True)
    for a, b in zip(full[0] + full[1], rec[0] + rec[1]):
        assert np.array_equal(a, b)
    for ga, gb_ in zip(full[2], rec[2]):
        for k in ga:
            assert np.array_equal(ga[k], gb_[k]), k
    compare(shape, rec, oracle_run(shape, params, xs, dys))
    e = 2 if dtype == "bf16" else 4
    T, H, F = shape.tokens, shape.hidden, shape.ffn
    saved = B.gpt_stage_stash_bytes(B.make_cfg(shape)) - B.gpt_stage_stash_bytes(B.make_cfg(rshape))
    assert saved == shape.n_layers * (2 * T * H + T * F) * e
    # level 2: the stash keeps only every layer's input; the backward phase runs the layer's
    # forward again.  Same bits again (decoupled: the forward of micro-batch 1 has overwritten
    # the forward workspace before the backward of micro-batch 0 re-runs its layers).
    xshape = shape.with_(recompute=2)
    only_x = gpu_run(xshape, params, xs, dys, decoupled=True)
    for a, b in zip(full[0] + full[1], only_x[0] + only_x[1]):
        assert np.array_equal(a, b)
    for ga, gb_ in zip(full[2], only_x[2]):
        for k in ga:
            assert np.array_equal(ga[k], gb_[k]), k
    res = 4   # the residual stream is fp32 in both storage types
    assert B.gpt_stage_stash_bytes(B.make_cfg(xshape)) == shape.n_layers * T * H * res
    if dtype == "bf16":
        f16 = gpu_run(shape.with_(recompute=2, hidden=256, ffn=512, fwd_fp16=True), params, xs, dys, decoupled=True)
        f16_ref = gpu_run(shape.with_(fwd_fp16=True), params, xs, dys, decoupled=True)
        for a, b in zip(f16[0] + f16[1], f16_ref[0] + f16_ref[1]):
            assert np.array_equal(a, b)
        for ga, gb_ in zip(f16[2], f16_ref[2]):
            for k in ga:
                assert np.array_equal(ga[k], gb_[k]), k


def test_stage_calls_can_be_captured_in_a_hip_graph():
    """The stage calls only enqueue kernels (and device-to-device copies) on the given stream and
    allocate nothing, so a forward + backward can be captured once and replayed.  Every replay --
    with the program's own eager work and synchronisations in between, and new inputs copied into
    the captured buffers -- must give the bits of the eager call.  The gradient buffer is cleared
    inside the graph by a fill kernel (not a memset node)."""
    shape = W[1].with_(name="bf16_graph", n_layers=2, hidden=256, n_heads=4, head_dim=64, ffn=512,
                       seq=128, batch=2, bias_std=0.02, ln_jitter=0.1)
    print(f"[case] hip graph {shape}", flush=True)
    params, xs, dys = _inputs(shape, n_mb=3)
    bufs = B.StageBuffers(shape)
    bufs.load_params(params)
    p = bufs.params()
    x_s, dy_s, y_s, dx_s = (bufs.act() for _ in range(4))       # the captured call's buffers
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):                              # warm-up outside capture
        B.gpt_stage_fwd_bwd(p, x_s, dy_s, bufs.stash[0], y_s, dx_s, bufs.dparams)
    torch.cuda.current_stream().wait_stream(side)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        bufs.dparams.zero_()
        B.gpt_stage_fwd_bwd(p, x_s, dy_s, bufs.stash[0], y_s, dx_s, bufs.dparams)
    for m in range(3):
        x_d, dy_d = B.to_device(xs[m], shape.dtype), B.to_device(dys[m], shape.dtype)
        # eager reference on separate buffers (also the "program's own work" between replays)
        ref = gpu_run(shape, params, [xs[m]], [dys[m]])
        torch.cuda.synchronize()
        x_s.copy_(x_d)
        dy_s.copy_(dy_d)
        graph.replay()
        torch.cuda.synchronize()
        assert np.array_equal(B.to_host(y_s), ref[0][0]) and np.array_equal(B.to_host(dx_s), ref[1][0]), m
        for ga, gb in zip(bufs.read_grads(), ref[2]):
            for k in ga:
                assert np.array_equal(ga[k], gb[k]), (m, k)
