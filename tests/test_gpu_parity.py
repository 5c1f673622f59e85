"""GPU parity tests: the HIP path, called through the C ABI, against the CPU
oracle on the same seeded inputs.  Protocol and tolerances: tests/parity.py."""
import numpy as np
import pytest
import torch

from synth_inputs import CONFIGS, SwitchShape, make_inputs

pytestmark = pytest.mark.gpu


def _dev():
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    return "cuda:0"


def _report(name, errs):
    print("\n[parity] %s: %s" % (name, {k: (("%.2e" % v) if isinstance(v, float) else v)
                                        for k, v in errs.items()}), flush=True)


# ----------------------------------------------------------------- fp32 path
def test_tiny_fp32_full_parity():
    from parity import compare_full
    s = CONFIGS["tiny"]
    inp = make_inputs(s, _dev())
    errs, gpu, fwd, _ = compare_full(s, inp, d_aux=1.0)
    _report("tiny", errs)
    assert fwd["capacity"] == 80


@pytest.mark.parametrize("T,d,f,E,cf,bias", [
    (300, 20, 36, 3, 0.7, True),      # ragged everything, drops, router bias
    (1000, 64, 128, 8, 1.0, False),   # several token blocks
    (64, 32, 64, 1, 1.0, False),      # single expert: dense FFN, gate 1
    (257, 16, 32, 5, 4.0, False),     # no drops
])
def test_fp32_shapes_full_parity(T, d, f, E, cf, bias):
    from parity import compare_full
    s = SwitchShape("t", T, d, f, E, cf, dtype="f32", zipf_bias=bias, seed_index=31)
    inp = make_inputs(s, _dev())
    errs, gpu, fwd, _ = compare_full(s, inp, d_aux=0.7)
    _report("fp32 %s" % ((T, d, f, E, cf, bias),), errs)
    if E == 1:
        assert np.all(gpu["gate"] == 1.0)
        assert np.abs(gpu["dW_r"]).max() == 0.0


# ----------------------------------------------------------------- bf16 path
@pytest.mark.parametrize("T,d,f,E,cf,bias", [
    (2000, 264, 520, 5, 1.5, False),   # 3 ragged token tiles, K tail (264 = 4*64 + 8), ragged p tiles
    (4096, 128, 256, 16, 1.0, True),   # Zipf bias: overflow and empty experts
    (1024, 64, 64, 1, 1.0, False),     # single expert, 4 full token tiles
    (777, 72, 136, 7, 0.5, False),     # heavy dropping, odd sizes
    (3000, 512, 768, 4, 1.25, False),  # several k steps and 3 x 2 p tiles
])
@pytest.mark.parametrize("in_gemm", [False, True])   # dispatch / combine as passes, or inside the GEMMs
def test_bf16_shapes_full_parity(T, d, f, E, cf, bias, in_gemm):
    from parity import compare_full
    s = SwitchShape("t", T, d, f, E, cf, dtype="bf16", zipf_bias=bias, seed_index=41,
                    fused_dispatch=in_gemm)
    inp = make_inputs(s, _dev())
    errs, gpu, fwd, _ = compare_full(s, inp, d_aux=1.0)
    _report("bf16 %s%s" % ((T, d, f, E, cf, bias), ", in the GEMMs" if in_gemm else ""), errs)
    if bias:
        assert fwd["dropped"].sum() > 0 and (fwd["expert_counts"] == 0).any()


@pytest.mark.parametrize("dtype,d,f,E", [
    ("bf16", 392, 72, 10), ("bf16", 136, 72, 60), ("bf16", 768, 136, 128), ("bf16", 264, 72, 200),
    ("f32", 132, 68, 10), ("f32", 392, 72, 60), ("f32", 392, 36, 128), ("f32", 64, 256, 4)])
def test_a_tokens_results_do_not_depend_on_the_batch(dtype, d, f, E):
    """A logit is one chain of sums over d, whatever the number of tokens has chosen as blocks, and so is an
    fp32 product, whatever tile: the first tokens of a large batch by themselves get the same bits."""
    from paper_2101_03961_amd.layer import SwitchLayer
    T, few = 40000, 150
    inp = make_inputs(SwitchShape("t", T, d, f, E, 4.0, dtype=dtype, seed_index=61), _dev())
    got = []
    for n, cf in ((T, 4.0), (few, float(E))):   # room for all tokens
        layer = SwitchLayer(n, d, f, E, cf, 0.01, dtype, _dev(), want_logits=True)
        x, dy = inp["x"][:n].contiguous(), inp["dy"][:n].contiguous()
        out = dict(layer.forward(x, inp["W_r"], inp["W_in"], inp["W_out"]))
        assert not out["dropped"].any()
        if dtype == "f32":
            out["dx"] = layer.backward(dy, x, inp["W_r"], inp["W_in"], inp["W_out"], d_aux=0.0)["dx"]
        got.append({k: out[k][:few].clone() for k in
                    ("router_logits", "expert_index") + (("gate", "y", "dx") if dtype == "f32" else ())})
    for k in got[0]:
        assert torch.equal(got[0][k], got[1][k]), k


@pytest.mark.parametrize("T,d,f,E,cf,likes", [
    (2400, 264, 904, 120, 1.25, "all"),    # two rounds of tiles, one k step, ragged in both dimensions
    (9000, 264, 760, 80, 1.25, "all"),     # two or three k steps
    (2400, 264, 904, 120, 4.0, "first"),   # experts of 80 tokens beside many without any
    (2500, 264, 904, 250, 4.0, "all"),     # E no multiple of the XCDs; four rounds of tiles:
    (2500, 264, 904, 250, 4.0, "first"),   # ... with tokens, then without, several in a row
    (2500, 264, 904, 250, 4.0, "last"),    # ... without tokens, then with
])
def test_weight_gradients_of_persistent_blocks(T, d, f, E, cf, likes):
    """Sizes that take the 384 x 256 and 256 x 384 tiles of gemm_wgrad.hip (listed in tests/test_launches.py)."""
    from parity import compare_full
    s = SwitchShape("t", T, d, f, E, cf, dtype="bf16", zipf_bias=likes != "all", seed_index=47)
    inp = make_inputs(s, _dev())
    if likes == "last":
        inp["b_r"] = inp["b_r"].flip(0).contiguous()
    errs, gpu, fwd, _ = compare_full(s, inp, d_aux=1.0)
    _report("persistent weight gradients %s" % ((T, d, f, E, cf, likes),), errs)
    empty = fwd["expert_counts"] == 0
    if E == 250 and likes != "all":   # a block's tiles lie about 64 experts apart
        assert empty[64:][:64].all() if likes == "first" else empty[:192].all()
        assert not empty[0 if likes == "first" else -1]


@pytest.mark.parametrize("T,cf,bias", [(500, 4.0, False), (2400, 1.25, False), (2400, 4.0, True)])
def test_large_weight_gradients_with_shared_lines(T, cf, bias):
    """Rows that share 128-byte lines, more than 512 MB: both gradients or the second one with guarded stores."""
    from parity import compare_sampled
    s = SwitchShape("t", T, 1080, 2408, 100, cf, dtype="bf16", zipf_bias=bias, seed_index=53)
    _report("shared lines %s" % ((T, cf, bias),), compare_sampled(s, make_inputs(s, _dev()), n_experts=3))


def test_bf16_without_slots():
    """Capacity 0 in a layer of many experts: zero outputs and zero weight gradients."""
    from parity import compare_full
    s = SwitchShape("t", 9000, 264, 760, 80, 0.007, dtype="bf16", seed_index=47)
    errs, gpu, fwd, _ = compare_full(s, make_inputs(s, _dev()), d_aux=1.0)
    _report("no slots", errs)
    assert fwd["capacity"] == 0 and fwd["dropped"].all()


@pytest.mark.parametrize("T,d,f,E,cf,ffn,bias", [
    (5000, 520, 776, 24, 1.25, "relu", False),   # tiles of 128 x 128, gradients of 256 x 128, ragged in all of them
    (3100, 264, 776, 11, 1.25, "geglu", True),   # 96 x 128 and 128 x 128, experts without tokens
    (500, 136, 520, 13, 2.0, "relu", False),     # 32 x 128 and 128 x 128
])
def test_three_backward_products_in_one_launch(T, d, f, E, cf, ffn, bias):
    from parity import compare_full
    s = SwitchShape("t", T, d, f, E, cf, dtype="bf16", zipf_bias=bias, seed_index=59, ffn=ffn)
    errs, _, _, _ = compare_full(s, make_inputs(s, _dev()), d_aux=1.0)
    _report("three products %s" % ((T, d, f, E, cf, ffn, bias),), errs)


@pytest.mark.parametrize("dtype,T,d,f,E,cf,n,jit,bias", [
    ("bf16", 1, 8, 8, 1, 4.0, 1, 0.0, True), ("bf16", 65, 72, 136, 65, 8.0, 1, 0.0, True),   # edges of 64 x 64 x 32
    ("bf16", 4160, 136, 264, 130, 1.25, 2, 0.0, True), ("f32", 97, 68, 132, 3, 1.0, 1, 0.0, True),
    ("f32", 4100, 132, 68, 64, 1.25, 4, 0.1, False), ("f32", 2100, 20, 36, 256, 2.0, 1, 0.0, True),
    # near the static scratch's limit: a launch of their own, in memory of the experts' gradients or beside it, or few parts
    ("bf16", 1050, 512, 2600, 16, 2.0, 1, 0.1, False), ("bf16", 1050, 512, 2600, 16, 2.0, 1, 0.0, True),
    ("f32", 1127, 568, 488, 139, 2.0, 1, 0.0, True), ("bf16", 713, 3456, 656, 42, 1.0, 1, 0.1, True)])
def test_router_weight_gradient_beside_the_experts(dtype, T, d, f, E, cf, n, jit, bias):
    """Its parts in blocks of the experts' launches, twice over on one forward pass."""
    from parity import compare_full
    s = SwitchShape("t", T, d, f, E, cf, dtype=dtype, zipf_bias=bias, seed_index=67, n_groups=n, jitter_eps=jit,
                    noise_seed=3)
    inp = make_inputs(s, _dev())
    errs, gpu, _, _ = compare_full(s, inp, d_aux=1.0)
    _report("router weight gradient %s" % ((dtype, T, d, f, E, cf, n, jit),), errs)
    from paper_2101_03961_amd.layer import SwitchLayer
    layer = SwitchLayer(T, d, f, E, cf, s.alpha, dtype, _dev(), n_groups=n, jitter_eps=jit, seed=3)
    args = (inp["x"], inp["W_r"], inp["W_in"], inp["W_out"], inp["b_r"])
    layer.forward(*args)
    layer.alloc_grads(with_bias=inp["b_r"] is not None)
    first = {k: v.clone() for k, v in layer.backward(inp["dy"], *args).items() if v is not None}
    again = layer.backward(inp["dy"], *args)
    assert all(torch.equal(first[k], again[k]) for k in first)


def router_gradient_error(SwitchLayer, T, d, E, dtype="f32", **kw):
    """dW_r of the load-balancing loss alone (dy = 0) against 64 bits: relative error, 2-norm."""
    gen = torch.Generator(device=_dev()).manual_seed(83)
    rand = lambda *size: torch.randn(size, generator=gen, device=_dev())
    x, W_r = rand(T, d), rand(d, E) * 0.002
    W_in, W_out = rand(E, d, 8), rand(E, 8, d)
    layer = SwitchLayer(T, d, 8, E, 1.0, 0.01, dtype, _dev(), **kw)
    args = (x, W_r, W_in, W_out)
    counts = layer.forward(*args)["expert_counts"].double()
    got = layer.backward(torch.zeros_like(x), *args)["dW_r"].double()
    p = torch.softmax(x.double() @ W_r.double(), 1)
    dp = (counts - T / E) * (0.01 * E / T ** 2)
    want = x.double().t() @ (p * (dp - (p * dp).sum(1, keepdim=True)))
    return float((got - want).norm() / want.norm())


def test_router_weight_gradient_sums_in_short_chains():
    """Few parts of many tokens (their memory is limited).  With terms of random sign a chain of n fp32 sums is off by
    2^-24 sqrt(n / 6) of its result: 2.8e-7 for 128 tokens, 1.0e-7 for the sum of the 16 chains of a part; one chain of
    2016 would be off by 1.1e-6."""
    from paper_2101_03961_amd.layer import SwitchLayer
    error = router_gradient_error(SwitchLayer, 30000, 8192, 32)
    _report("router weight gradient in chains", {"dW_r": error})
    assert error <= 4e-7


@pytest.mark.parametrize("T,d,E,n", [(1, 8, 3, 1), (65, 72, 32, 1), (130, 40, 33, 1), (1000, 264, 64, 2), (700, 136, 128, 1),
                                     (515, 72, 130, 1), (300, 264, 256, 4),
                                     (70, 1032, 132, 1), (333, 1160, 256, 1)])   # planes of x * m
@pytest.mark.parametrize("fused", [False, True])
def test_bf16_tokens_with_jitter_in_the_one_kernel_router(T, d, E, n, fused):
    """fp32 products of x * m, forward and backward, beside the other route; the logits to fp32 rounding."""
    from parity import compare_full
    s = SwitchShape("t", T // n * n, d, 72, E, 1.25, dtype="bf16", zipf_bias=E % 4 != 0, seed_index=73, n_groups=n,
                    jitter_eps=0.1, noise_seed=11, fused_dispatch=fused)
    errs, _, _, _ = compare_full(s, make_inputs(s, _dev()), d_aux=1.0)
    _report("jitter %s" % ((T, d, E, n, fused),), errs)


@pytest.mark.parametrize("T,d,f,E,cf,n,rate,ffn,rounds", [
    (12000, 264, 1544, 64, 1.0, 1, 0.0, "relu", 0),     # 256 x 384, one row tile per expert, ragged both ways
    (16000, 264, 1544, 60, 1.25, 2, 0.1, "relu", 0),    # 320 x 256, two row tiles, groups, dropout
    (20000, 520, 1544, 40, 1.25, 1, 0.0, "geglu", 0),   # every product
    (20000, 520, 1544, 40, 1.0, 1, 0.0, "relu", 2),     # re-routing fills more experts than the router asked for
])
def test_few_large_tiles_in_pieces(T, d, f, E, cf, n, rate, ffn, rounds):
    """A collapsed router leaves one or two of many experts with tokens: their large tiles run in pieces."""
    from parity import compare_full
    s = SwitchShape("t", T, d, f, E, cf, dtype="bf16", zipf_bias=True, seed_index=53, n_groups=n, expert_dropout=rate,
                    ffn=ffn, ntlb_rounds=rounds, noise_seed=3)
    errs, gpu, fwd, _ = compare_full(s, make_inputs(s, _dev()), d_aux=1.0)
    _report("few tiles %s" % ((T, d, f, E, cf, n, rate, ffn, rounds),), errs)
    assert rounds or (fwd["expert_counts"] > 0).sum() <= 8


@pytest.mark.parametrize("d,E,cf,tiles", [
    (136, 8, 1.96875, 63), (136, 8, 2.0, 64), (200, 8, 2.0, 65), (136, 4, 2.0, 128)])   # (200: two experts)
def test_many_row_tiles_of_one_expert(d, E, cf, tiles):
    """Second forward GEMM and first data gradient with one column tile of 256 x 256, so that a collapsed router
    leaves as many tiles as its favourite has rows of 256: up to 64 run in pieces, which all have to be counted."""
    from parity import compare_full
    s = SwitchShape("t", 65536, d, 264, E, cf, dtype="bf16", zipf_bias=True, seed_index=71)
    errs, gpu, fwd, _ = compare_full(s, make_inputs(s, _dev()), d_aux=1.0)
    _report("row tiles %s" % ((d, E, cf),), errs)
    kept = np.minimum(fwd["expert_counts"], fwd["capacity"])
    assert (-(-kept // 256)).sum() == tiles


@pytest.mark.parametrize("T,d,f,E,cf,n,bias,ffn,rate,rounds", [
    (2000, 264, 520, 5, 1.5, 1, False, "relu", 0.0, 0),    # ragged tiles everywhere
    (4096, 128, 256, 16, 1.0, 2, True, "relu", 0.1, 1),    # groups, skew, dropout, re-routing
    (3000, 512, 768, 4, 1.25, 1, False, "geglu", 0.0, 0),  # gated-GELU experts
])
def test_bf16_dispatch_inside_the_gemms_agrees_with_the_passes(T, d, f, E, cf, n, bias, ffn, rate, rounds):
    """Dispatch and combine as passes of their own (the default) and inside the GEMMs (on
    request): each against the oracle, and against each other to rounding."""
    from parity import compare_full
    s = SwitchShape("t", T, d, f, E, cf, dtype="bf16", zipf_bias=bias, seed_index=43, n_groups=n,
                    ffn=ffn, expert_dropout=rate, noise_seed=5, ntlb_rounds=rounds)
    inp = make_inputs(s, _dev())
    errs, sep, _, _ = compare_full(s, inp, d_aux=0.9)
    _report("bf16 separate passes %s" % ((T, d, f, E, cf, n, ffn),), errs)
    errs, fused, _, _ = compare_full(s.with_(fused_dispatch=True), inp, d_aux=0.9)
    _report("bf16 inside the GEMMs %s" % ((T, d, f, E, cf, n, ffn),), errs)
    for k in ("expert_index", "gate", "position_in_expert", "dropped", "expert_counts", "aux_loss",
              "router_logits"):
        assert np.array_equal(sep[k], fused[k]), k
    for k in ("y", "dx", "dW_in", "dW_out"):
        a, b = sep[k].astype(np.float64), fused[k].astype(np.float64)
        assert np.linalg.norm(a - b) <= 1e-2 * np.linalg.norm(b), k


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_capacity_zero_everything_dropped(dtype):
    from parity import compare_full
    s = SwitchShape("t", 5, 64, 64, 8, 1.0, dtype=dtype, seed_index=51)
    inp = make_inputs(s, _dev())
    errs, gpu, fwd, bwd = compare_full(s, inp)
    assert fwd["capacity"] == 0 and gpu["dropped"].all()
    assert np.all(gpu["y"] == 0) and np.all(gpu["dW_in"] == 0) and np.all(gpu["dW_out"] == 0)
    assert np.abs(gpu["dx"]).max() > 0          # the auxiliary loss still reaches x


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("T,E,cf", [
    (1, 4, 4.0),     # a single token, capacity 1
    (7, 16, 4.0),    # more experts than tokens, capacity 1
    (7, 16, 1.0),    # ... and capacity floor(7/16) = 0
    (255, 3, 1.0),   # one short token block
    (257, 3, 1.0),   # one token into the second block
])
def test_few_tokens(dtype, T, E, cf):
    from parity import compare_full
    s = SwitchShape("t", T, 64, 72, E, cf, dtype=dtype, seed_index=54)
    inp = make_inputs(s, _dev())
    # With a handful of kept tokens all of dW_r and db_r is a few gate gradients
    # <dy_t, o_t> times fixed vectors: their error is measured against the scale of those dot
    # products' terms (parity.router_grad_scales), as for every other case.
    errs, gpu, fwd, _ = compare_full(s, inp, d_aux=0.3)
    _report("few tokens %s %s" % (dtype, (T, E, cf)), errs)
    assert fwd["capacity"] == int(np.floor(T / E * cf))


@pytest.mark.parametrize("T,d,f,E,cf", [
    (1500, 96, 64, 128, 2.0),    # the widest router the matrix-core kernel takes
    (1500, 96, 64, 124, 2.0),    # four experts short of it
    (3000, 64, 64, 132, 1.0),    # one step wider: vector-ALU router, bf16 tokens
    (3000, 64, 64, 256, 1.0),    # two experts per lane in the softmax kernels
    (2048, 72, 64, 126, 1.0),    # E not a multiple of 4: vector-ALU router
])
def test_bf16_router_widths(T, d, f, E, cf):
    from parity import compare_full
    s = SwitchShape("t", T, d, f, E, cf, dtype="bf16", seed_index=55)
    inp = make_inputs(s, _dev())
    errs, gpu, fwd, _ = compare_full(s, inp, d_aux=1.0)
    _report("bf16 router E=%d" % E, errs)


@pytest.mark.parametrize("dtype,T,d,f,E,cf,n", [
    ("f32", 600, 32, 48, 4, 1.0, 2),       # 300 tokens per group: blocks of 256 + 44
    ("f32", 90, 16, 24, 3, 0.9, 5),        # groups smaller than a token block
    ("bf16", 4096, 128, 256, 16, 1.0, 8),  # groups of two full blocks
    ("bf16", 3000, 96, 136, 12, 1.25, 3),  # 1000 tokens per group
    ("bf16", 2100, 64, 72, 7, 0.5, 7),     # heavy dropping in every group, vector-ALU router
])
def test_routing_groups(dtype, T, d, f, E, cf, n):
    """Capacity, positions and the loss fractions per routing group; shared experts."""
    from parity import compare_full
    s = SwitchShape("t", T, d, f, E, cf, dtype=dtype, seed_index=57, n_groups=n)
    inp = make_inputs(s, _dev())
    if dtype == "bf16":   # also with dispatch / combine inside the GEMMs
        errs = compare_full(s.with_(fused_dispatch=True), inp, d_aux=0.8)[0]
        _report("groups %s, in the GEMMs" % ((dtype, T, E, cf, n),), errs)
    errs, gpu, fwd, _ = compare_full(s, inp, d_aux=0.8)
    _report("groups %s" % ((dtype, T, E, cf, n),), errs)
    assert fwd["capacity"] == int(np.floor(T / n / E * cf))
    # positions restart in every group
    Tg = T // n
    first = np.array([np.flatnonzero(gpu["expert_index"][g * Tg:(g + 1) * Tg] ==
                                     gpu["expert_index"][g * Tg])[0] for g in range(n)])
    assert np.all(first == 0) and np.all(gpu["position_in_expert"][::Tg] == 0)


def test_routing_groups_full_size():
    """Switch-Base shape as eight routing groups (capacity 64 per expert and group)."""
    from parity import compare_sampled
    s = CONFIGS["base_cf1.0"].with_(n_groups=8)
    inp = make_inputs(s, _dev())
    errs = compare_sampled(s, inp, n_experts=2, n_tokens=24)
    _report("base_cf1.0 x 8 groups", errs)


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_empty_batch(dtype):
    """T = 0: counts and loss zero, weight gradients zero, nothing else touched."""
    import torch
    import oracle
    from paper_2101_03961_amd.layer import SwitchLayer
    s = SwitchShape("t", 0, 64, 72, 4, 1.0, dtype=dtype, seed_index=56)
    inp = make_inputs(s, _dev())
    layer = SwitchLayer(0, 64, 72, 4, 1.0, s.alpha, dtype, device=_dev())
    layer.expert_counts.fill_(7)
    layer.aux_loss.fill_(7.0)
    layer.forward(inp["x"], inp["W_r"], inp["W_in"], inp["W_out"], None)
    layer.alloc_grads(with_bias=True)
    for g in (layer.dW_r, layer.db_r, layer.dW_in, layer.dW_out):
        g.fill_(1.0)
    layer.backward(inp["dy"], inp["x"], inp["W_r"], inp["W_in"], inp["W_out"], None, 1.0)
    torch.cuda.synchronize()
    to_np = lambda t: t.float().cpu().numpy()
    ref = oracle.forward(to_np(inp["x"]), to_np(inp["W_r"]), to_np(inp["W_in"]),
                         to_np(inp["W_out"]), 1.0, s.alpha)
    assert ref["aux_loss"] == 0.0 and ref["capacity"] == 0 and ref["y"].shape == (0, 64)
    assert float(layer.aux_loss[0]) == ref["aux_loss"]
    assert layer.expert_counts.tolist() == ref["expert_counts"].tolist() == [0, 0, 0, 0]
    for g in (layer.dW_r, layer.db_r, layer.dW_in, layer.dW_out):
        assert float(g.float().abs().max()) == 0.0


def test_exact_ties_go_to_expert_zero():
    from parity import run_gpu
    s = SwitchShape("t", 300, 64, 64, 6, 1.0, dtype="bf16", seed_index=52)
    inp = make_inputs(s, _dev())
    inp["W_r"].zero_()
    _, gpu = run_gpu(s, inp, backward=False)
    assert np.all(gpu["expert_index"] == 0)
    assert np.all(gpu["gate"] == np.float32(1.0) / np.float32(6.0))
    assert gpu["expert_counts"].tolist() == [300, 0, 0, 0, 0, 0]
    assert np.array_equal(gpu["position_in_expert"], np.arange(300))
    assert np.array_equal(gpu["dropped"], (np.arange(300) >= 50).astype(np.uint8))
    assert abs(float(gpu["aux_loss"][0]) - 0.01) < 1e-7      # P uniform => loss = alpha


@pytest.mark.parametrize("in_gemm", [False, True])
def test_run_to_run_determinism(in_gemm):
    from parity import run_gpu
    s = SwitchShape("t", 5000, 256, 512, 12, 1.0, dtype="bf16", seed_index=53, fused_dispatch=in_gemm)
    inp = make_inputs(s, _dev())
    _, a = run_gpu(s, inp)
    _, b = run_gpu(s, inp)
    for k in a:
        assert np.array_equal(a[k], b[k]), k


@pytest.mark.parametrize("dtype,in_gemm", [("f32", False), ("bf16", False), ("bf16", True)])
def test_scaling_and_expert_permutation_properties(dtype, in_gemm):
    """Properties of the GPU path alone.  Doubling W_out doubles y exactly (a power of two
    changes no rounding).  Renumbering the experts (columns of W_r, blocks of W_in / W_out)
    renumbers expert_index and the counts and leaves every token's slot; gate and output move
    only by the rounding of the softmax sum taken in another order (and what follows from it)."""
    from parity import run_gpu
    s = SwitchShape("t", 3000, 128, 264, 12, 1.0, dtype=dtype, seed_index=92, fused_dispatch=in_gemm)
    inp = make_inputs(s, _dev())
    _, a = run_gpu(s, inp, backward=False)
    doubled = dict(inp, W_out=inp["W_out"] * 2)
    _, b = run_gpu(s, doubled, backward=False)
    assert np.array_equal(b["y"], 2 * a["y"])
    for k in ("expert_index", "gate", "dropped", "position_in_expert", "aux_loss"):
        assert np.array_equal(a[k], b[k]), k
    perm = torch.randperm(s.E, generator=torch.Generator().manual_seed(5)).to(_dev())
    shuffled = dict(inp, W_r=inp["W_r"][:, perm].contiguous(), W_in=inp["W_in"][perm].contiguous(),
                    W_out=inp["W_out"][perm].contiguous())
    _, c = run_gpu(s, shuffled, backward=False)
    p = perm.cpu().numpy()
    assert np.array_equal(p[c["expert_index"]], a["expert_index"])
    assert np.array_equal(c["expert_counts"], a["expert_counts"][p])
    for k in ("dropped", "position_in_expert"):
        assert np.array_equal(a[k], c[k]), k
    np.testing.assert_allclose(c["gate"], a["gate"], rtol=5e-7, atol=0)
    # one rounding step of the storage type; with the combine inside the GEMMs also: the gate
    # scales the hidden activations before they are rounded, so a gate that moves by one fp32 ulp
    # flips the rounding of a few of them: a row may move by a small share of its RMS
    ulp = 2.0 ** -7 if dtype == "bf16" else 1e-6
    rms = np.sqrt(np.mean(a["y"].astype(np.float64) ** 2, axis=1, keepdims=True))
    floor = 2.0 ** -9 * rms if in_gemm else 1e-30
    assert np.all(np.abs(c["y"].astype(np.float64) - a["y"]) <= ulp * np.abs(a["y"]) + floor)
    assert abs(float(a["aux_loss"][0]) - float(c["aux_loss"][0])) <= 1e-6 * abs(float(a["aux_loss"][0]))


@pytest.mark.parametrize("dtype,T,d,f,E,cf,n", [
    ("bf16", 16384, 64, 64, 4096, 2.0, 1),  # the largest expert count the library takes
    ("f32", 3000, 32, 48, 1000, 3.0, 1),
    ("bf16", 6000, 72, 64, 513, 1.0, 2),    # nine experts per lane in the softmax kernels
])
def test_many_experts(dtype, T, d, f, E, cf, n):
    from parity import compare_full
    s = SwitchShape("t", T, d, f, E, cf, dtype=dtype, seed_index=59, n_groups=n)
    inp = make_inputs(s, _dev())
    errs, gpu, fwd, _ = compare_full(s, inp, d_aux=0.5)
    _report("E=%d" % E, errs)


@pytest.mark.parametrize("T,d,f,E,cf,n,bias,eps,rounds", [
    (4096, 128, 72, 256, 2.0, 1, False, 0.0, 0),      # two full expert tiles
    (3000, 200, 64, 200, 1.0, 2, True, 0.0, 1),       # second tile partly filled, ragged d
    (2048, 776, 64, 1024, 4.0, 1, False, 0.01, 0),    # eight tiles, jittered input planes
    (5000, 96, 64, 132, 1.5, 1, True, 0.0, 2),        # four experts in the second tile
])
def test_bf16_router_on_matrix_cores_beyond_128_experts(T, d, f, E, cf, n, bias, eps, rounds):
    """More than 128 experts (a multiple of 4): the logits come from the matrix-core kernel, one
    tile of 128 experts per block, softmax and the rest from the vector-ALU path's kernel."""
    from parity import compare_full
    s = SwitchShape("t", T, d, f, E, cf, dtype="bf16", seed_index=62, n_groups=n, zipf_bias=bias,
                    jitter_eps=eps, noise_seed=17, ntlb_rounds=rounds)
    errs = compare_full(s, make_inputs(s, _dev()), d_aux=0.5)[0]
    _report("bf16 router, E=%d" % E, errs)


def test_fp32_long_reduction():
    """One expert holding 17 576 tokens: each weight-gradient element is a sum over all of them,
    which the fp32 path takes in two levels (a single fp32 chain drifts past 1e-5 here)."""
    from parity import compare_full
    s = SwitchShape("t", 17576, 292, 152, 1, 1.25, dtype="f32", seed_index=61, n_groups=8)
    errs = compare_full(s, make_inputs(s, _dev()), d_aux=0.5)[0]
    _report("fp32, 17576 tokens in one expert", errs)
    assert errs["dW_in"] < 2e-6 and errs["dW_out"] < 2e-6


def test_random_shapes():
    """Seeded sweep over token counts, widths, expert counts, capacity factors, group counts
    and both storage types: every tile edge and kernel variant at sizes the full oracle takes
    a fraction of a second for."""
    from parity import compare_full
    rng = np.random.default_rng(20210111)
    for case in range(36):
        dtype = "bf16" if rng.random() < 0.75 else "f32"
        mult = 8 if dtype == "bf16" else 4
        E = int(rng.choice([1, 2, 3, 4, 6, 8, 12, 16, 20, 32, 64]))
        n = int(rng.choice([1, 1, 1, 2, 3, 4]))
        T = int(rng.integers(200, 1400)) * n
        hi_d, hi_f = (640, 800) if dtype == "bf16" else (400, 400)
        d = int(rng.integers(32 // mult, hi_d // mult)) * mult
        f = int(rng.integers(32 // mult, hi_f // mult)) * mult
        cf = float(rng.choice([0.7, 1.0, 1.25, 2.0, 8.0]))
        in_gemm = dtype == "bf16" and case % 2 == 1
        s = SwitchShape("t", T, d, f, E, cf, dtype=dtype, seed_index=300 + case, n_groups=n,
                        fused_dispatch=in_gemm)
        print("[random shape %d] %s T=%d d=%d f=%d E=%d cf=%g groups=%d in_gemm=%d" %
              (case, dtype, T, d, f, E, cf, n, in_gemm), flush=True)
        inp = make_inputs(s, _dev())
        compare_full(s, inp, d_aux=0.5)


def test_random_shapes_with_options():
    """The same sweep with the optional parts switched on at random: gated-GELU experts,
    expert dropout, input jitter, re-routing stages, router bias."""
    from parity import compare_full
    rng = np.random.default_rng(20210112)
    for case in range(30):
        dtype = "bf16" if rng.random() < 0.7 else "f32"
        mult = 8 if dtype == "bf16" else 4
        E = int(rng.choice([2, 3, 4, 6, 8, 16, 32, 128]))
        n = int(rng.choice([1, 1, 2, 4]))
        T = int(rng.integers(300, 1400)) * n
        hi_d, hi_f = (520, 400) if dtype == "bf16" else (300, 200)
        d = int(rng.integers(32 // mult, hi_d // mult)) * mult
        f = int(rng.integers(32 // mult, hi_f // mult)) * mult
        cf = float(rng.choice([0.7, 1.0, 1.25, 2.0]))
        ffn = "geglu" if rng.random() < 0.5 else "relu"
        rate = float(rng.choice([0.0, 0.1, 0.4]))
        eps = float(rng.choice([0.0, 0.0, 0.01, 0.1]))
        rounds = int(rng.choice([0, 0, 1, 2, 4]))
        bias = bool(rng.random() < 0.4)
        s = SwitchShape("t", T, d, f, E, cf, dtype=dtype, seed_index=400 + case, n_groups=n,
                        ffn=ffn, expert_dropout=rate, jitter_eps=eps,
                        noise_seed=int(rng.integers(0, 2 ** 62)), ntlb_rounds=rounds, zipf_bias=bias,
                        fused_dispatch=dtype == "bf16" and case % 2 == 0)
        print("[random options %d] %s T=%d d=%d f=%d E=%d cf=%g groups=%d %s drop=%g jitter=%g "
              "stages=%d bias=%d in_gemm=%d" % (case, dtype, T, d, f, E, cf, n, ffn, rate, eps, rounds,
                                                bias, s.fused_dispatch), flush=True)
        inp = make_inputs(s, _dev())
        compare_full(s, inp, d_aux=0.5)


def test_relu_decision_at_a_zero_preactivation():
    """In this seeded case one pre-activation is -7.5e-9 in fp64 (RMS of its row: 1) and the
    fp32 sum of the same exact products comes out positive: the unit's gate is a coin flip,
    the protocol follows the GPU's decision for that one (token, unit) pair."""
    from parity import compare_full
    s = SwitchShape("t", 1206, 208, 712, 1, 2.0, dtype="bf16", seed_index=152)
    inp = make_inputs(s, _dev())
    errs, gpu, fwd, _ = compare_full(s, inp, d_aux=0.5)
    _report("zero pre-activation", errs)
    import oracle
    npi = {k: (None if v is None else v.float().cpu().numpy()) for k, v in inp.items()}
    near = oracle.hidden_near_zero(npi["x"], npi["W_in"], fwd["expert_index"], fwd["dropped"], 1e-6)
    assert (252, 515) in [(t, j) for t, j, _ in near] and len(near) <= 4, near
    assert all(abs(h) < 1e-5 for _, _, h in near)


@pytest.mark.parametrize("options", [
    {},
    dict(fused_dispatch=True),
    dict(ffn="geglu", expert_dropout=0.1, jitter_eps=0.01, noise_seed=3, ntlb_rounds=2),
    dict(ffn="geglu", expert_dropout=0.1, jitter_eps=0.01, noise_seed=3, ntlb_rounds=2,
         fused_dispatch=True),
])
def test_step_can_be_captured_in_a_graph(options):
    """Forward + backward recorded once and replayed: every replay, with eager work and
    synchronisation between them, reproduces the eager result bit for bit (the library launches
    only kernels: no allocation, no memset node, no host synchronisation)."""
    import torch
    from paper_2101_03961_amd.layer import SwitchLayer
    s = SwitchShape("t", 3000, 256, 512, 12, 1.0, dtype="bf16", seed_index=58, n_groups=2,
                    **options)
    inp = make_inputs(s, _dev())
    layer = SwitchLayer(s.T, s.d_model, s.d_ff, s.E, s.capacity_factor, s.alpha, s.dtype,
                        device=_dev(), n_groups=s.n_groups, ffn=s.ffn,
                        expert_dropout=s.expert_dropout, jitter_eps=s.jitter_eps,
                        seed=s.noise_seed, ntlb_rounds=s.ntlb_rounds, fused_dispatch=s.fused_dispatch)
    layer.alloc_grads(with_bias=False)
    names = ("y", "dx", "dW_r", "dW_in", "dW_out", "aux_loss", "expert_counts", "gate", "dropped")

    def step():
        layer.forward(inp["x"], inp["W_r"], inp["W_in"], inp["W_out"], None)
        layer.backward(inp["dy"], inp["x"], inp["W_r"], inp["W_in"], inp["W_out"], None, 1.0)

    step()
    torch.cuda.synchronize()
    eager = {k: getattr(layer, k).clone() for k in names}
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        step()
    torch.cuda.current_stream().wait_stream(side)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        step()
    for _ in range(3):
        for k in names:
            getattr(layer, k).fill_(3)
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        for k in names:
            assert torch.equal(getattr(layer, k), eager[k]), k
        assert float(layer.y.float().abs().sum()) > 0   # eager work between replays


# ------------------------------------------- training-time noise (Sec. 2.4, App. C)
@pytest.mark.parametrize("dtype,T,d,f,E,cf,n,bias,rate,eps,seed", [
    ("f32", 700, 96, 200, 6, 1.0, 1, False, 0.1, 0.01, 0x123456789ABC),     # both, 48-bit seed
    ("f32", 1024, 64, 136, 8, 0.75, 4, True, 0.4, 0.0, 5),                  # dropout only, groups
    ("f32", 515, 72, 64, 5, 2.0, 1, False, 0.0, 0.25, 2 ** 63 + 11),        # jitter only
    ("bf16", 1500, 256, 520, 6, 1.25, 1, False, 0.4, 0.1, 7),
    ("bf16", 2048, 128, 264, 128, 1.5, 2, True, 0.0, 0.01, 99),             # would take the MFMA router
    ("bf16", 3000, 776, 304, 16, 1.0, 3, False, 0.1, 0.0, 2 ** 40),         # MFMA router + dropout
])
def test_training_noise(dtype, T, d, f, E, cf, n, bias, rate, eps, seed):
    from parity import compare_full
    s = SwitchShape("t", T, d, f, E, cf, dtype=dtype, seed_index=70, n_groups=n, zipf_bias=bias,
                    expert_dropout=rate, jitter_eps=eps, noise_seed=seed)
    inp = make_inputs(s, _dev())
    if dtype == "bf16":   # also with dispatch / combine inside the GEMMs
        errs = compare_full(s.with_(fused_dispatch=True), inp, d_aux=0.8)[0]
        _report("noise %s rate %.2f eps %.2f, in the GEMMs" % (dtype, rate, eps), errs)
    errs, gpu, fwd, _ = compare_full(s, inp, d_aux=0.8)
    _report("noise %s rate %.2f eps %.2f" % (dtype, rate, eps), errs)
    # the noise did something: outputs differ from the noise-free layer's
    _, plain = run_gpu_plain(s, inp)
    assert not np.array_equal(plain["y"], gpu["y"])
    if eps > 0:
        assert not np.array_equal(plain["router_logits"], gpu["router_logits"])
    else:
        assert np.array_equal(plain["router_logits"], gpu["router_logits"])
        assert np.array_equal(plain["expert_index"], gpu["expert_index"])


def run_gpu_plain(s, inp):
    from parity import run_gpu
    return run_gpu(s.with_(expert_dropout=0.0, jitter_eps=0.0), inp, backward=False)


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_training_noise_depends_on_the_seed_only(dtype):
    from parity import run_gpu
    s = SwitchShape("t", 2000, 128, 256, 8, 1.25, dtype=dtype, seed_index=71, expert_dropout=0.3,
                    jitter_eps=0.05, noise_seed=1)
    inp = make_inputs(s, _dev())
    _, a = run_gpu(s, inp)
    _, b = run_gpu(s, inp)
    _, c = run_gpu(s.with_(noise_seed=2), inp)
    _, hi = run_gpu(s.with_(noise_seed=1 + (1 << 32)), inp)
    for k in a:
        assert np.array_equal(a[k], b[k]), k
    for other in (c, hi):
        assert not np.array_equal(a["y"], other["y"])
        assert not np.array_equal(a["router_logits"], other["router_logits"])
    # zero rates: the seed is not looked at
    z0 = run_gpu(s.with_(expert_dropout=0.0, jitter_eps=0.0, noise_seed=0), inp)[1]
    z1 = run_gpu(s.with_(expert_dropout=0.0, jitter_eps=0.0, noise_seed=12345), inp)[1]
    for k in z0:
        assert np.array_equal(z0[k], z1[k]), k
    # dropout keeps about 1 - rate of the active hidden units: dW_out rows of dropped units
    # are zero for a token; count exact zeros of y instead -- none expected for kept tokens
    kept = a["dropped"] == 0
    assert np.all(np.abs(a["y"][kept]).sum(axis=1) > 0)


def test_training_noise_full_size_sampled():
    """Switch-Base shape with the fine-tuning expert dropout of Table 4 and jitter."""
    from parity import compare_sampled
    s = CONFIGS["base_cf1.25"].with_(expert_dropout=0.4, jitter_eps=0.01, noise_seed=20210111)
    inp = make_inputs(s, _dev())
    errs = compare_sampled(s, inp, n_experts=2, n_tokens=24)
    _report("base_cf1.25 + noise", errs)


# ------------------------------------------- gated-GELU experts (model tables, FFN_GEGLU)
@pytest.mark.parametrize("dtype,T,d,f,E,cf,n,rate,eps", [
    ("f32", 700, 96, 100, 6, 1.0, 1, 0.0, 0.0),
    ("f32", 1024, 64, 36, 8, 0.75, 4, 0.25, 0.05),
    ("bf16", 1500, 256, 520, 6, 1.25, 1, 0.0, 0.0),     # ragged tiles in every GEMM
    ("bf16", 4096, 128, 264, 16, 1.0, 2, 0.1, 0.0),
    ("bf16", 3000, 776, 128, 5, 2.0, 1, 0.0, 0.01),
    ("bf16", 600, 64, 8, 3, 1.0, 1, 0.0, 0.0),          # the narrowest hidden layer
])
def test_geglu_experts(dtype, T, d, f, E, cf, n, rate, eps):
    from parity import compare_full
    s = SwitchShape("t", T, d, f, E, cf, dtype=dtype, seed_index=80, n_groups=n, ffn="geglu",
                    expert_dropout=rate, jitter_eps=eps, noise_seed=31)
    inp = make_inputs(s, _dev())
    assert inp["W_in"].shape == (E, d, 2 * f)
    if dtype == "bf16":   # also with dispatch / combine inside the GEMMs
        errs = compare_full(s.with_(fused_dispatch=True), inp, d_aux=0.8)[0]
        _report("geglu %s f=%d, in the GEMMs" % (dtype, f), errs)
    errs, gpu, fwd, _ = compare_full(s, inp, d_aux=0.8)
    assert gpu["dW_in"].shape == (E, d, 2 * f)
    _report("geglu %s f=%d" % (dtype, f), errs)


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_geglu_capacity_zero_and_empty_batch(dtype):
    from parity import run_gpu
    from paper_2101_03961_amd.layer import SwitchLayer
    s = SwitchShape("t", 64, 64, 72, 128, 1.0, dtype=dtype, seed_index=81, ffn="geglu")  # capacity 0
    inp = make_inputs(s, _dev())
    _, gpu = run_gpu(s, inp)
    assert np.all(gpu["dropped"] == 1) and np.all(gpu["y"] == 0)
    assert np.all(gpu["dW_in"] == 0) and np.all(gpu["dW_out"] == 0)
    layer = SwitchLayer(0, 64, 72, 4, 1.0, s.alpha, dtype, device=_dev(), ffn="geglu")
    e = lambda *shape: torch.empty(shape, dtype=layer.act, device=_dev())
    W_r = torch.zeros((64, 4), device=_dev())
    layer.forward(e(0, 64), W_r, e(4, 64, 144), e(4, 72, 64))
    layer.alloc_grads(with_bias=False)
    layer.dW_in.fill_(1.0)
    layer.dW_out.fill_(1.0)
    g = layer.backward(e(0, 64), e(0, 64), W_r, e(4, 64, 144), e(4, 72, 64))
    torch.cuda.synchronize()
    assert g["dW_in"].shape == (4, 64, 144) and float(g["dW_in"].float().abs().sum()) == 0.0
    assert float(g["dW_out"].float().abs().sum()) == 0.0


def test_layer_refuses_wrong_weight_shape():
    """The ReLU layout handed to a gated-GELU layer must not reach the kernels."""
    from paper_2101_03961_amd.layer import SwitchLayer
    s = SwitchShape("t", 256, 64, 72, 4, 1.0, dtype="bf16", seed_index=82)
    inp = make_inputs(s, _dev())
    layer = SwitchLayer(s.T, s.d_model, s.d_ff, s.E, 1.0, s.alpha, "bf16", device=_dev(), ffn="geglu")
    with pytest.raises(ValueError):
        layer.forward(inp["x"], inp["W_r"], inp["W_in"], inp["W_out"])


def test_geglu_switch_base_sampled():
    from parity import compare_sampled
    s = CONFIGS["base_geglu"]
    inp = make_inputs(s, _dev())
    errs = compare_sampled(s, inp, n_experts=2, n_tokens=24)
    _report("base_geglu", errs)


# ------------------------------------------- No-Token-Left-Behind (App. B)
@pytest.mark.parametrize("dtype,T,d,f,E,cf,n,bias,rounds,ffn", [
    ("f32", 700, 64, 96, 6, 1.0, 1, True, 1, "relu"),
    ("f32", 1024, 64, 40, 8, 0.75, 4, True, 3, "geglu"),
    ("bf16", 3000, 128, 264, 16, 1.0, 1, False, 1, "relu"),     # MFMA router, mild overflow
    ("bf16", 4096, 128, 264, 128, 1.0, 2, True, 2, "relu"),     # heavy skew, 128 experts
    ("bf16", 2500, 72, 64, 513, 2.0, 1, False, 2, "relu"),      # nine experts per lane, ragged
    ("f32", 600, 32, 32, 3, 1.0, 1, True, 16, "relu"),          # more rounds than experts
])
def test_no_token_left_behind(dtype, T, d, f, E, cf, n, bias, rounds, ffn):
    from parity import compare_full, run_gpu
    s = SwitchShape("t", T, d, f, E, cf, dtype=dtype, seed_index=90, n_groups=n, zipf_bias=bias,
                    ntlb_rounds=rounds, ffn=ffn)
    inp = make_inputs(s, _dev())
    if dtype == "bf16":   # also with dispatch / combine inside the GEMMs
        errs = compare_full(s.with_(fused_dispatch=True), inp, d_aux=0.7)[0]
        _report("ntlb %s E=%d rounds=%d, in the GEMMs" % (dtype, E, rounds), errs)
    errs, gpu, fwd, _ = compare_full(s, inp, d_aux=0.7)
    _, plain = run_gpu(s.with_(ntlb_rounds=0), inp, backward=False)
    rescued = int(plain["dropped"].sum()) - int(gpu["dropped"].sum())
    errs["rescued"], errs["still_dropped"] = rescued, int(gpu["dropped"].sum())
    _report("ntlb %s E=%d rounds=%d" % (dtype, E, rounds), errs)
    assert rescued > 0
    # tokens that had a slot keep it; the loss and the counts do not change
    k1 = plain["dropped"] == 0
    assert np.array_equal(plain["expert_index"][k1], gpu["expert_index"][k1])
    assert np.array_equal(plain["position_in_expert"][k1], gpu["position_in_expert"][k1])
    assert np.array_equal(plain["expert_counts"], gpu["expert_counts"])
    assert np.array_equal(plain["aux_loss"], gpu["aux_loss"])
    # no (group, expert) pair exceeds its capacity
    kept = gpu["dropped"] == 0
    key = (np.arange(T) // (T // n))[kept] * E + gpu["expert_index"][kept]
    assert np.bincount(key, minlength=n * E).max() <= fwd["capacity"]


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_groups_of_two_tokens(dtype):
    """The smallest routing groups: two tokens each, one slot per (group, expert); with a
    re-routing stage the second token of a pair that collides moves to the other expert."""
    from parity import compare_full
    s = SwitchShape("t", 2048, 64, 72, 2, 1.0, dtype=dtype, seed_index=91, n_groups=1024)
    inp = make_inputs(s, _dev())
    errs, gpu, fwd, _ = compare_full(s, inp, d_aux=0.6)
    assert fwd["capacity"] == 1 and 0 < gpu["dropped"].sum() < 1024
    _report("groups of two", errs)
    errs, gpu2, _, _ = compare_full(s.with_(ntlb_rounds=1), inp, d_aux=0.6)
    assert gpu2["dropped"].sum() == 0          # two tokens, two experts with one slot each
    _report("groups of two + re-routing", errs)


def test_no_token_left_behind_full_size():
    from parity import compare_sampled
    s = CONFIGS["base_cf1.0"].with_(ntlb_rounds=2)
    inp = make_inputs(s, _dev())
    errs = compare_sampled(s, inp, n_experts=2, n_tokens=24)
    _report("base_cf1.0 + 2 re-routing stages", errs)


# ------------------------------------------- full sizes
# The metric's own workload (Switch-Base, capacity factor 1.0: 65 536 tokens, 128 experts)
# against the complete fp64 oracle, forward and backward: every row of y and dx, every expert's
# weight gradients, the router's.  The oracle takes the experts sixteen at a time (the GEMMs'
# eight tile ranges); each range is a test of its own, so that the run reports every twenty
# seconds instead of staying silent for minutes, and the router's gradients, which need every
# range, come last.
_BASE_FULL = {}


def _base_full():
    from parity import FullByExperts
    if "run" not in _BASE_FULL:
        s = CONFIGS["base_cf1.0"]
        _BASE_FULL["run"] = FullByExperts(s, make_inputs(s, _dev()), n_chunks=8, d_aux=1.0)
    return _BASE_FULL["run"]


@pytest.mark.parametrize("c", range(8))
def test_switch_base_full_oracle_parity_experts(c):
    run = _base_full()
    print("\n" + run.chunk(c), flush=True)
    assert run.fwd["capacity"] == 512 and int(run.fwd["dropped"].sum()) > 0


def test_switch_base_full_oracle_parity_router():
    run = _base_full()
    if len(run.done) < run.n_chunks:
        pytest.skip("needs every expert range of test_switch_base_full_oracle_parity_experts")
    errs = run.router()
    _BASE_FULL.clear()          # the tensors are large
    _report("base_cf1.0, full oracle", errs)


@pytest.mark.parametrize("name,n_experts", [
    ("base_cf1.25", 18), ("base_zipf", 18), ("large", 12), ("c_share", 6), ("base_e256", 12),
])
def test_full_size_sampled_parity(name, n_experts):
    """The other full-size workloads: all outputs finite, routing on every token, and the
    experts at the edges of the GEMMs' tile ranges (plus the fullest and the emptiest) against
    the oracle."""
    from parity import compare_sampled
    s = CONFIGS[name]
    inp = make_inputs(s, _dev())
    errs = compare_sampled(s, inp, n_experts=n_experts, n_tokens=24)
    _report(name, errs)


@pytest.mark.parametrize("name,n_experts", [("base_cf1.0", 18), ("base_cf1.25", 10)])
def test_full_size_sampled_parity_inside_the_gemms(name, n_experts):
    """The full-size workloads with dispatch and combine inside the GEMMs (gathered operand
    loads, scattered output rows, at 3072+ tiles per launch): same checks as above."""
    from parity import compare_sampled
    s = CONFIGS[name].with_(fused_dispatch=True)
    inp = make_inputs(s, _dev())
    errs = compare_sampled(s, inp, n_experts=n_experts, n_tokens=24)
    _report(name + ", in the GEMMs", errs)


def test_xxl_sampled_parity():
    """Largest shape: the first, the last, the fullest and the emptiest expert plus single
    tokens; the fp64 oracle needs about 0.5 GFLOP per token here."""
    from parity import compare_sampled
    s = CONFIGS["xxl"]
    inp = make_inputs(s, _dev())
    errs = compare_sampled(s, inp, n_experts=4, n_tokens=16)
    _report("xxl", errs)


# Tile shapes of the one-tile-per-block GEMMs, each at ragged rows, columns and depth; the comments
# name the tiles of the first- and second-layer products (rows x columns).
@pytest.mark.parametrize("T,d,f,E,cf,rate,ffn", [
    (200, 264, 520, 12, 1.5, 0.0, "relu"),      # 32 x 128 both; weight gradients: few large tiles
    (33, 72, 136, 4, 1.0, 0.3, "relu"),         # ... a handful of rows, one k step
    (1900, 264, 776, 40, 1.25, 0.0, "relu"),    # 96 x 128 and 32 x 128
    (2000, 264, 1032, 40, 2.0, 0.2, "relu"),    # dropout in both masked epilogues
    (5003, 392, 1000, 10, 1.25, 0.0, "relu"),   # 128 x 128 and 96 x 128
    (6000, 200, 2312, 16, 1.0, 0.1, "relu"),    # 256-row tiles; two per expert, the second short
    (9000, 72, 2312, 16, 1.25, 0.0, "relu"),    # 256 x 384, three row tiles, one and a bit k steps
    (2500, 136, 520, 40, 1.0, 0.0, "geglu"),    # plain products, first layer twice as wide
])
def test_row_tiles_full_parity(T, d, f, E, cf, rate, ffn):
    from parity import compare_full
    s = SwitchShape("t", T, d, f, E, cf, dtype="bf16", seed_index=45, expert_dropout=rate, noise_seed=9,
                    ffn=ffn)
    inp = make_inputs(s, _dev())
    errs, gpu, fwd, _ = compare_full(s, inp, d_aux=1.0)
    _report("row tiles %s" % ((T, d, f, E, cf, rate, ffn),), errs)


# fp32 GEMMs on the matrix cores: edges of 64-row / 64- and 128-column tiles, k tails, two-level sums
@pytest.mark.parametrize("T,d,f,E,cf,rate,ffn", [
    (900, 20, 1028, 128, 2.0, 0.0, "relu"),    # wide tiles (many of them), k = 20 and a k tail of 4
    (700, 68, 132, 5, 1.0, 0.25, "relu"),      # one column group past a tile, third row tile short
    (600, 516, 36, 2, 1.25, 0.0, "geglu"),     # k past two flushes of the running sum
])
def test_fp32_matrix_core_tiles(T, d, f, E, cf, rate, ffn):
    from parity import compare_full
    s = SwitchShape("t", T, d, f, E, cf, dtype="f32", seed_index=46, expert_dropout=rate, noise_seed=3,
                    ffn=ffn)
    inp = make_inputs(s, _dev())
    errs, gpu, fwd, _ = compare_full(s, inp, d_aux=0.8)
    _report("fp32 tiles %s" % ((T, d, f, E, cf, rate, ffn),), errs)


# The FMA kernel with 64-bit addresses: slots x hidden units of an expert reach 2 GB (room for a million slots,
# 50 tokens in them), all six products, the dropout epilogue
def test_fp32_beyond_one_buffer_descriptor():
    from parity import compare_full
    s = SwitchShape("t", 101, 12, 516, 2, 20800.0, dtype="f32", seed_index=50, expert_dropout=0.25, noise_seed=3)
    inp = make_inputs(s, _dev())
    errs, gpu, fwd, _ = compare_full(s, inp, d_aux=0.8)
    _report("fp32 2 GB", errs)
    assert fwd["capacity"] * 516 * 4 >= 1 << 31


# Router forward in one kernel and the assign kernel: expert tiles of 32 with and without 16-byte
# weight loads, token blocks of 64 (and 128 from 32768 tokens on) with remainders, block prefix sums
# inside the assign kernel (up to 128 token blocks) and by the scan kernel, groups that end inside a block
@pytest.mark.parametrize("dtype,T,d,E,cf,n", [
    ("bf16", 63, 72, 3, 1.0, 1), ("bf16", 65, 40, 30, 2.0, 1), ("bf16", 129, 136, 33, 1.0, 3),
    ("bf16", 1000, 776, 60, 1.25, 1), ("bf16", 8192, 64, 126, 1.0, 1), ("bf16", 8193, 64, 128, 1.0, 1),
    ("bf16", 2085, 72, 132, 1.0, 5), ("bf16", 700, 200, 256, 1.5, 1), ("bf16", 32768, 16, 31, 1.0, 8),
    ("bf16", 32779, 40, 64, 1.0, 1), ("bf16", 33001, 16, 100, 0.8, 1), ("bf16", 34000, 8, 250, 1.0, 2),
    ("f32", 66, 20, 5, 1.0, 1), ("f32", 1030, 132, 36, 1.25, 2), ("f32", 9000, 12, 128, 1.0, 1),
    ("f32", 500, 68, 201, 2.0, 1),
])
def test_router_forward_blocks(dtype, T, d, E, cf, n):
    from parity import compare_full
    s = SwitchShape("t", T, d, 24, E, cf, dtype=dtype, seed_index=47, n_groups=n)
    inp = make_inputs(s, _dev())
    errs, gpu, fwd, _ = compare_full(s, inp, d_aux=1.2)
    _report("router blocks %s" % ((dtype, T, d, E, cf, n),), errs)


# Router backward in one kernel: expert counts with and without 16-byte rows at each fragment count
# (32, 64, 128; with fp32 operands 256), token remainders of the 128-token blocks, column groups of 64 with
# remainders in one or several blocks, groups that end inside a block, bias sums, jitter on bf16 tokens
@pytest.mark.parametrize("dtype,T,d,E,cf,n,jit,bias", [
    ("bf16", 31, 8, 2, 1.0, 1, 0.0, True), ("bf16", 129, 72, 32, 1.0, 1, 0.0, True),
    ("bf16", 390, 136, 33, 1.0, 3, 0.0, True), ("bf16", 3000, 1032, 63, 1.25, 1, 0.0, False),
    ("bf16", 1025, 200, 128, 1.5, 1, 0.0, True), ("bf16", 2050, 328, 100, 1.0, 2, 0.05, True),
    ("f32", 1, 4, 3, 3.0, 1, 0.0, True), ("f32", 257, 132, 32, 1.0, 1, 0.1, True),
    ("f32", 640, 68, 62, 1.0, 5, 0.0, False), ("f32", 1000, 36, 256, 1.0, 1, 0.0, True),
    ("f32", 129, 100, 131, 2.0, 1, 0.0, True), ("bf16", 700, 104, 253, 1.0, 2, 0.0, True),
])
def test_router_backward_blocks(dtype, T, d, E, cf, n, jit, bias):
    from parity import compare_full
    s = SwitchShape("t", T, d, 24, E, cf, dtype=dtype, seed_index=48, n_groups=n, jitter_eps=jit, noise_seed=4,
                    zipf_bias=bias)
    inp = make_inputs(s, _dev())
    errs, gpu, fwd, _ = compare_full(s, inp, d_aux=1.3)
    _report("router backward %s" % ((dtype, T, d, E, cf, n, jit, bias),), errs)


# Router gradients from fp32 operands: fp32 tokens, and bf16 tokens where the expert count is no multiple
# of 4.  At capacity 0 they are the loss's alone and exact up to fp32 arithmetic: each of their terms sees
# a few roundings of 2^-24 (logit, exponential, quotient, product, sums of 64 in a chain), 2 .. 3e-7 of the
# norm together.  Operands of two bf16 terms, 2^-18 off, would show 1.6e-6.
@pytest.mark.parametrize("dtype,E", [("bf16", 3), ("bf16", 10), ("bf16", 33), ("bf16", 126), ("bf16", 130),
                                     ("bf16", 250), ("f32", 64), ("f32", 201)])
def test_router_gradients_keep_fp32_operands(dtype, E):
    from paper_2101_03961_amd.layer import SwitchLayer
    T, d = 1500, 200
    inp = make_inputs(SwitchShape("t", T, d, 24, E, 1e-4, dtype=dtype, seed_index=49), _dev())
    layer = SwitchLayer(T, d, 24, E, 1e-4, 0.01, dtype, _dev())
    args = (inp["x"], inp["W_r"], inp["W_in"], inp["W_out"])
    counts = layer.forward(*args)["expert_counts"].cpu().double()
    grads = layer.backward(inp["dy"], *args, d_aux=2.0)
    x, W = inp["x"].cpu().double(), inp["W_r"].cpu().double()
    p = torch.softmax(x @ W, 1)
    dp = 2.0 * 0.01 * E / T ** 2 * counts
    dl = p * (dp - (p * dp).sum(1, keepdim=True))
    for name, want in (("dW_r", x.T @ dl), ("db_r", dl.sum(0))):
        err = float((grads[name].cpu().double() - want).norm() / want.norm())
        _report("fp32 router operands %s %s" % ((dtype, E), name), {"err": err})
        if name == "dW_r":
            assert err < 2.0 ** -20
    want = dl @ W.T
    err = float((grads["dx"].cpu().double() - want).norm() / want.norm())
    # one rounding to the tokens' type: at most half a unit, 2^-9 of the value in bf16
    assert err < (2.0 ** -9 if dtype == "bf16" else 2.0 ** -20)


@pytest.mark.parametrize("dtype,T,d,E,jitter", [("f32", 70, 72, 8, 0.0), ("bf16", 70, 72, 8, 0.0), ("bf16", 70, 72, 300, 0.0),
                                                ("bf16", 70, 1032, 132, 0.1), ("bf16", 16400, 64, 128, 0.1)])
def test_token_without_a_largest_logit(dtype, T, d, E, jitter):
    """Not a number in a token: it goes to expert 0, like equal logits, and no other token's results change."""
    from paper_2101_03961_amd.layer import SwitchLayer
    gen = torch.Generator(device=_dev()).manual_seed(89)
    act = torch.bfloat16 if dtype == "bf16" else torch.float32
    rand = lambda *size: torch.randn(size, generator=gen, device=_dev())
    x, dy, W_r = rand(T, d).to(act), rand(T, d).to(act), rand(d, E)
    W_in, W_out = (rand(E, d, 16) * 0.1).to(act), (rand(E, 16, d) * 0.1).to(act)
    others = torch.arange(T, device=_dev()) != 37
    outs = []
    for value in (0.0, float("nan")):
        x[37] = value
        layer = SwitchLayer(T, d, 16, E, 4.0, 0.01, dtype, _dev(), jitter_eps=jitter, seed=5)
        fwd = {k: v.clone() for k, v in layer.forward(x, W_r, W_in, W_out).items() if v is not None}
        dx = layer.backward(dy, x, W_r, W_in, W_out)["dx"].clone()
        assert fwd["expert_index"][37] == 0
        outs.append([fwd["expert_index"], fwd["expert_counts"], fwd["y"][others], dx[others]])
    assert all(torch.equal(a, b) for a, b in zip(*outs))
