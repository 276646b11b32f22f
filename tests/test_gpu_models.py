"""GPU parity, end to end: every served architecture through the C ABI (submit at a priority ->
pinned H2D -> kernel sequence -> D2H -> record) against the CPU oracle on the same seeded inputs."""
import numpy as np
import pytest

import synth
from oracle import models as omodels
from parity import check_kernel, check_logits

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    import paper_2604_28175_amd as strait
    c = strait.Context(device=0, n_hp=1, n_lp=1, n_copy=2)
    c.S = strait
    yield c
    c.close()


def run_cnn(ctx, md, x, fwd, prio, what):
    S = ctx.S
    m = ctx.load(synth.pack(md), max_batch=x.shape[0], n_instances=1)
    try:
        out, rec = m.infer(x, prio=prio)
        ref = fwd(md.tensors, x)
        err, scale, ties = check_logits(out["logits"], ref.logits, out["top1"], what)
        assert np.abs(out["probs"] - ref.probs).max() <= 2e-2
        assert np.abs(out["probs"].sum(-1) - 1).max() < 1e-4
        assert rec.batch == x.shape[0] and rec.priority == prio
        assert rec.h2d_ms > 0 and rec.kernel_ms > 0 and rec.total_ms >= rec.kernel_ms
        assert rec.t_enqueue_ns <= rec.t_issued_ns <= rec.t_done_ns
        print(f"{what}: max|err| {err:.3e} of scale {scale:.3e} ({err / scale:.2e}), ties {ties}, kernels {rec.kernel_ms:.3f} ms")
        return m, out, ref
    except Exception:
        m.free()
        raise


def test_tiny_cnn_config(ctx):
    md = synth.tiny_cnn(synth.SEEDS[synth.ARCH_TINY_CNN])
    x = synth.default_image_batch(md, 4, synth.SEEDS[synth.ARCH_TINY_CNN] + 4)
    m, out, ref = run_cnn(ctx, md, x, omodels.tiny_cnn_forward, ctx.S.PRIO_HIGH, "tiny CNN b4")
    # zero input: zero biases -> logits exactly 0, uniform probabilities
    z, _ = m.infer(np.zeros_like(x))
    assert not z["logits"].any() and np.allclose(z["probs"], 0.1, atol=1e-6) and not z["top1"].any()
    m.free()


@pytest.mark.parametrize("hw,batch", [(64, 5), (224, 2)])
def test_resnet50(ctx, hw, batch):
    md = synth.resnet50(synth.SEEDS[synth.ARCH_RESNET50], hw=hw)
    x = synth.default_image_batch(md, batch, synth.SEEDS[synth.ARCH_RESNET50] + batch)
    m, out, ref = run_cnn(ctx, md, x, omodels.resnet50_forward, ctx.S.PRIO_HIGH, f"ResNet-50 {hw}px b{batch}")
    m.free()


def test_resnet50_layers_and_batch_independence(ctx):
    """Every layer's activation against the oracle's (catches wiring errors that cancel in the
    logits), and sample i of a batch equals the same image run alone."""
    md = synth.resnet50(3, hw=64)
    x = synth.default_image_batch(md, 3, 8)
    m = ctx.load(synth.pack(md), max_batch=3, n_instances=1)
    ref = omodels.resnet50_forward(md.tensors, x, keep=True)
    m.copy_in(0, ctx.S.PRIO_LOW, x)
    names = {}
    for i, li in enumerate(m.layers()):
        names[li.name.decode()] = i
    checked = 0
    for lname, act in ref.trace.acts.items():
        key = lname.replace(".out", ".c3")       # the fused epilogue of c3 produces the block output
        if lname.endswith(".c3") or key not in names or lname in ("fc",):
            continue
        got = m.read_activation(0, names[key], 3).astype(np.float64).reshape(act.shape)
        check_kernel(got, act, f"layer {lname}", rel=2.0 ** -8, abs_rel=1e-2)
        checked += 1
    assert checked >= 40
    full, _ = m.infer(x, prio=ctx.S.PRIO_LOW)
    for i in range(3):
        one, _ = m.infer(x[i:i + 1], prio=ctx.S.PRIO_LOW)
        assert np.abs(one["logits"][0] - full["logits"][i]).max() <= 1e-3 * np.abs(full["logits"]).max()
        assert one["top1"][0] == full["top1"][i]
    m.free()


def test_resnet50_fused_block_seams_equal_separate_launches(ctx):
    """The closing 1x1 of a bottleneck and the opening 1x1 of the next one as one launch (forced at every size here,
    ragged tiles included) give the logits of the layer-by-layer plan bit for bit, and the oracle's within tolerance."""
    md = synth.resnet50(5)            # full size, six images: no layer of a fused pair is small enough to split its reduction
    x = synth.default_image_batch(md, 6, 9)
    m = ctx.load(synth.pack(md), max_batch=6, n_instances=1)
    try:
        ctx.set_proj_fusion(1 << 40)  # the first block's pair with its projection shortcut is not bit-identical: below
        ctx.set_pair_fusion(0)
        sep, _ = m.infer(x, prio=ctx.S.PRIO_HIGH)
        ctx.set_pair_fusion(1)
        fused, _ = m.infer(x, prio=ctx.S.PRIO_HIGH)
        names = [l.name.decode() for l in m.layers()]
        assert np.array_equal(sep["logits"], fused["logits"]) and np.array_equal(sep["top1"], fused["top1"])
        ref = omodels.resnet50_forward(md.tensors, x)
        check_logits(fused["logits"], ref.logits, fused["top1"], "ResNet-50 b6, fused seams")
        # intermediate activations read back through the fused path
        ref = omodels.resnet50_forward(md.tensors, x, keep=True)
        # (s1b0.c1 is computed inside the fused stem + pooling launch)
        for lname, key in (("s1b0.c1", "s1b0.c1"), ("s1b1.c1", "s1b1.c1"), ("s1b1.out", "s1b1.c3"), ("s1b2.out", "s1b2.c3"), ("s2b0.c1", "s2b0.c1")):
            got = m.read_activation(0, names.index(key), 6).astype(np.float64).reshape(ref.trace.acts[lname].shape)
            check_kernel(got, ref.trace.acts[lname], f"layer {lname}", rel=2.0 ** -8, abs_rel=1e-2)
        # the first block's closing 1x1, its projection shortcut and the next block's opening 1x1 as one launch: one
        # rounding fewer than the separate launches, so against the oracle only
        ctx.set_proj_fusion(1)
        proj, _ = m.infer(x, prio=ctx.S.PRIO_HIGH)
        check_logits(proj["logits"], ref.logits, proj["top1"], "ResNet-50 b6, projection in the fused seam")
        assert not np.array_equal(proj["logits"], fused["logits"])          # (the other path did run)
        for lname, key in (("s1b0.out", "s1b0.c3"), ("s1b1.c1", "s1b1.c1"), ("s1b1.out", "s1b1.c3")):
            got = m.read_activation(0, names.index(key), 6).astype(np.float64).reshape(ref.trace.acts[lname].shape)
            check_kernel(got, ref.trace.acts[lname], f"layer {lname} (projection fused)", rel=2.0 ** -8, abs_rel=1e-2)
    finally:
        ctx.set_pair_fusion(40000)
        ctx.set_proj_fusion(1)
        m.free()


@pytest.mark.parametrize("hw,batch", [(64, 5), (224, 2)])
def test_mobilenet_v2(ctx, hw, batch):
    md = synth.mobilenet_v2(synth.SEEDS[synth.ARCH_MOBILENETV2], hw=hw)
    x = synth.default_image_batch(md, batch, synth.SEEDS[synth.ARCH_MOBILENETV2] + batch)
    m, out, ref = run_cnn(ctx, md, x, omodels.mobilenet_v2_forward, ctx.S.PRIO_LOW, f"MobileNetV2 {hw}px b{batch}")
    m.free()


def test_mobilenet_v2_fused_expansions_equal_separate_launches(ctx):
    """At batch 6 every inverted residual block runs its expansion and its depthwise layer as one launch; the kernel takes the same arithmetic steps, so the whole network's output
    must be bit-identical with the fusion switched off, and the oracle's within tolerance."""
    md = synth.mobilenet_v2(synth.SEEDS[synth.ARCH_MOBILENETV2])
    x = synth.default_image_batch(md, 6, 99)
    m = ctx.load(synth.pack(md), max_batch=6, n_instances=1)
    try:
        ctx.set_pair_fusion(0)
        sep, _ = m.infer(x, prio=ctx.S.PRIO_LOW)
        ctx.set_pair_fusion(40000)
        fused, _ = m.infer(x, prio=ctx.S.PRIO_LOW)
        assert np.array_equal(sep["logits"], fused["logits"]) and np.array_equal(sep["top1"], fused["top1"])
        ref = omodels.mobilenet_v2_forward(md.tensors, x)
        check_logits(fused["logits"], ref.logits, fused["top1"], "MobileNetV2 b6, fused expansions")
    finally:
        ctx.set_pair_fusion(40000)
        m.free()


@pytest.mark.parametrize("batch,hw", [(12, 224), (33, 96), (40, 160)])
def test_mobilenet_v2_some_expansions_fused(ctx, batch, hw):
    """Sizes at which one launch is estimated to be faster for some of the blocks and two for the others: bit for bit what the
    network gives with the fusion switched off."""
    md = synth.mobilenet_v2(synth.SEEDS[synth.ARCH_MOBILENETV2], hw)
    x = synth.default_image_batch(md, batch, 98)
    m = ctx.load(synth.pack(md), max_batch=batch, n_instances=1)
    try:
        ctx.set_pair_fusion(0)
        sep, _ = m.infer(x, prio=ctx.S.PRIO_LOW)
        ctx.set_pair_fusion(40000)
        fused, _ = m.infer(x, prio=ctx.S.PRIO_LOW)
        assert np.array_equal(sep["logits"], fused["logits"]) and np.array_equal(sep["top1"], fused["top1"])
    finally:
        ctx.set_pair_fusion(40000)
        m.free()


def test_run_timed_gives_zero_for_layers_inside_another_launch(ctx):
    """Per-layer times: a layer that runs inside its predecessor's launch reads exactly 0, every launch a positive time."""
    md = synth.mobilenet_v2(synth.SEEDS[synth.ARCH_MOBILENETV2], hw=64)
    m = ctx.load(synth.pack(md), max_batch=4, n_instances=1)
    try:
        m.copy_in(0, ctx.S.PRIO_LOW, synth.default_image_batch(md, 4, 3))
        names = [l.name.decode() for l in m.layers()]
        ms = m.run_timed(0, ctx.S.PRIO_LOW, 4)
        inside = [n for n, t in zip(names, ms) if t == 0.0]
        assert inside == [f"b{i}.dw" for i in range(17)], inside   # behind its expansion; the first block's behind the stem
        assert all(t > 0.0 for n, t in zip(names, ms) if n not in inside)
        ctx.set_pair_fusion(0)
        assert all(t > 0.0 for t in m.run_timed(0, ctx.S.PRIO_LOW, 4))
    finally:
        ctx.set_pair_fusion(40000)
        m.free()


@pytest.mark.parametrize("kw,batch", [(dict(layers=2, hidden=128, heads=2, ffn=256, seq=64), 3),
                                      (dict(layers=2, hidden=128, heads=2, ffn=256, seq=48), 3),      # no multiple of the 32-row blocks
                                      (dict(layers=1, hidden=64, heads=1, ffn=128, seq=200), 2),      # more than 128 keys
                                      (dict(), 2)])
def test_encoder(ctx, kw, batch):
    md = synth.encoder(synth.SEEDS[synth.ARCH_ENCODER], **kw)
    x, vl = synth.token_batch(md, batch, synth.SEEDS[synth.ARCH_ENCODER] + batch, min_len=32)
    m = ctx.load(synth.pack(md), max_batch=batch, n_instances=1)
    out, rec = m.infer(x, vl, prio=ctx.S.PRIO_LOW)
    ref = omodels.encoder_forward(md.tensors, x, vl, md.hyper)
    scale = max(float(np.abs(ref.logits[b, :vl[b]]).max()) for b in range(batch))
    worst = 0.0
    for b in range(batch):
        L = int(vl[b])
        got = out["hidden"][b, :L].astype(np.float64)
        assert np.isfinite(got).all()
        worst = max(worst, float(np.abs(got - ref.logits[b, :L]).max()))
    assert worst <= 2e-2 * scale, f"encoder: max|err| {worst:.3e} > 2e-2 * {scale:.3e}"
    # top-1 of token 0 (same tie rule as the classifiers)
    check_logits(out["hidden"][:, 0, :], ref.logits[:, 0, :], out["top1"], "encoder token 0")
    print(f"encoder {md.hyper} b{batch}: max|err| {worst:.3e} of {scale:.3e}, kernels {rec.kernel_ms:.3f} ms")
    m.free()


@pytest.mark.parametrize("arch,kw,batch", [("encoder", dict(layers=3, hidden=128, heads=2, ffn=256, seq=40), 5),
                                           ("encoder", dict(layers=2, hidden=768, heads=12, ffn=3072, seq=128), 3),
                                           ("encoder", dict(layers=2, hidden=1024, heads=16, ffn=512, seq=33), 2),     # sixteen statistics a row
                                           ("encoder", dict(layers=2, hidden=1088, heads=17, ffn=256, seq=33), 2),     # one too many: not folded
                                           ("encoder", dict(layers=2, hidden=128, heads=2, ffn=200, seq=40), 2),       # FFN1 cannot take it in
                                           ("vit", dict(layers=3, hidden=192, heads=3, ffn=384), 3)])
def test_folded_layernorms(ctx, arch, kw, batch):
    """LayerNorms inside the products on their two sides against launches of their own; segments; every layer's own output; timing."""
    if arch == "encoder":
        md = synth.encoder(5, **kw)
        x, vl = synth.token_batch(md, batch, 7, min_len=20)
        ref = omodels.encoder_forward(md.tensors, x, vl, md.hyper, keep=True)
    else:
        md = synth.vit(5, hw=96, classes=50, **kw)
        x, vl = synth.default_image_batch(md, batch, 7), None
        ref = omodels.vit_forward(md.tensors, x, md.hyper, keep=True)
    key = "hidden" if arch == "encoder" else "logits"
    m = ctx.load(synth.pack(md), max_batch=batch, n_instances=1)
    rows = [slice(0, int(n)) for n in vl] if arch == "encoder" else [slice(None)] * batch
    try:
        got = m.infer(x, vl, prio=ctx.S.PRIO_LOW)[0][key]
        for b in range(batch):
            check_kernel(got[b][rows[b]], ref.logits[b][rows[b]], f"{arch} sample {b}", rel=2.0 ** -8, abs_rel=1e-2)
        ctx.set_lp_yield(1)                                  # every layer in a segment of its own
        assert np.array_equal(m.infer(x, vl, prio=ctx.S.PRIO_LOW)[0][key], got)
        ctx.set_lp_yield(3)
        assert np.array_equal(m.infer(x, vl, prio=ctx.S.PRIO_LOW)[0][key], got)
        ctx.set_lp_yield(0)
        ctx.set_pair_fusion(0)
        apart = m.infer(x, vl, prio=ctx.S.PRIO_LOW)[0][key]
        for b in range(batch):
            check_kernel(apart[b][rows[b]], got[b][rows[b]].astype(np.float64), f"{arch} sample {b} apart", rel=2.0 ** -8, abs_rel=1e-2)
        ctx.set_pair_fusion(40000)
        if vl is not None:
            m.copy_in(0, ctx.S.PRIO_LOW, x, vl)
        else:
            m.copy_in(0, ctx.S.PRIO_LOW, x)
        names = [li.name.decode() for li in m.layers()]
        checked = 0
        for i, nm in enumerate(names):
            if nm not in ref.trace.acts or not nm.startswith("l") or nm == f"l{kw['layers'] - 1}.ln2":      # (the last one is the output)
                continue
            act = ref.trace.acts[nm]
            a = m.read_activation(0, i, batch).astype(np.float64).reshape(act.shape)
            for b in range(batch):
                check_kernel(a[b][rows[b]], act[b][rows[b]], f"layer {nm}", rel=2.0 ** -8, abs_rel=1e-2)
            checked += 1
        assert checked >= 5 * kw["layers"] - 1
    finally:
        ctx.set_lp_yield(0)
        ctx.set_pair_fusion(40000)
        m.free()


@pytest.mark.parametrize("hidden,seq,batch,folds", [(1024, 35, 88, False), (1024, 32, 96, True), (832, 33, 125, False), (832, 32, 128, True), (768, 33, 125, True),   # one side and the other of 3072, 4096 rows
                                                    (512, 32, 2, False), (512, 65, 1, True), (1024, 64, 1, False), (448, 32, 2, True)])            # 64 and 65
def test_layernorms_are_folded_where_that_is_no_slower(ctx, hidden, seq, batch, folds):
    """The layer-by-layer plan's bytes where they are not."""
    md = synth.encoder(5, layers=2, hidden=hidden, heads=hidden // 64, ffn=256, seq=seq)
    x, vl = synth.token_batch(md, batch, 7, min_len=20)
    m = ctx.load(synth.pack(md), max_batch=batch, n_instances=1)
    try:
        got = m.infer(x, vl, prio=ctx.S.PRIO_LOW)[0]["hidden"]
        ctx.set_pair_fusion(0)
        apart = m.infer(x, vl, prio=ctx.S.PRIO_LOW)[0]["hidden"]
        assert np.array_equal(got, apart) != folds
        check_kernel(got[0][:int(vl[0])], apart[0][:int(vl[0])].astype(np.float64), "folded and apart", rel=2.0 ** -8, abs_rel=1e-2)
    finally:
        ctx.set_pair_fusion(40000)
        m.free()


@pytest.mark.parametrize("norms", [("l0.ln1", "l0.ln2", "l1.ln1", "l1.ln2", "l2.ln1"), ("l0.ln1", "l1.ln2"), ("l0.ln2",)])
def test_layernorms_whose_folded_weights_leave_the_normal_range(ctx, norms):
    """gamma of 2^-14 takes fp16 weights below the normal range: such a LayerNorm stays apart, beside folded ones."""
    md = synth.encoder(5, layers=3, hidden=128, heads=2, ffn=256, seq=40)
    for k in norms:
        md.tensors[k + ".g"] = np.full_like(md.tensors[k + ".g"], 2.0 ** -14)
    x, vl = synth.token_batch(md, 3, 7, min_len=20)
    ref = omodels.encoder_forward(md.tensors, x, vl, md.hyper).logits
    m = ctx.load(synth.pack(md), max_batch=3, n_instances=1)
    try:
        got = m.infer(x, vl, prio=ctx.S.PRIO_LOW)[0]["hidden"]
        ctx.set_pair_fusion(0)
        apart = m.infer(x, vl, prio=ctx.S.PRIO_LOW)[0]["hidden"]
        if len(norms) == 5:                              # every LayerNorm that could be folded
            assert np.array_equal(got, apart)
        for b in range(3):
            n = int(vl[b])
            check_kernel(got[b][:n], ref[b][:n], f"sample {b}", rel=2.0 ** -8, abs_rel=1e-2)
            check_kernel(apart[b][:n], ref[b][:n], f"sample {b} apart", rel=2.0 ** -8, abs_rel=1e-2)
    finally:
        ctx.set_pair_fusion(40000)
        m.free()


def test_a_model_that_fits_without_folded_layernorms_only(ctx):
    """With memory left for one set of weights and half of the second: loaded, and its results are those of the layer-by-layer plan, bit for bit; with
    less than one set it is refused, and with all memory back it is loaded as ever."""
    import torch
    S = ctx.S
    layers, hidden, ffn = 8, 1024, 4096
    md = synth.encoder(5, layers=layers, hidden=hidden, heads=16, ffn=ffn, seq=64)
    blob = synth.pack(md)
    second = layers * (3 * hidden + ffn) * hidden * 2      # Q, K, V and the first feed-forward product once more
    x, vl = synth.token_batch(md, 2, 7, min_len=20)

    def free():
        torch.cuda.synchronize()
        return torch.cuda.mem_get_info()[0]
    before = free()
    m = ctx.load(blob, max_batch=2, n_instances=1)
    both = before - free()
    assert both > len(blob) + second // 2                  # (it is folded)
    folded = m.infer(x, vl)[0]["hidden"]
    ctx.set_pair_fusion(0)
    apart = m.infer(x, vl)[0]["hidden"]
    ctx.set_pair_fusion(40000)
    m.free()
    assert not np.array_equal(folded, apart)
    filler = []
    try:
        for left, fits in ((both - second // 2, True), (len(blob) // 2, False)):
            for _ in range(8):                             # (what the driver calls free can grow with the first large allocation)
                if free() - left >= 4 << 20:
                    filler.append(torch.empty(free() - left, dtype=torch.uint8, device="cuda"))
            if abs(free() - left) >= 16 << 20:
                pytest.skip("something else takes or gives back the GPU's memory")
            if fits:
                m = ctx.load(blob, max_batch=2, n_instances=1)
                got = m.infer(x, vl)[0]["hidden"]
                m.free()
                assert np.array_equal(got, apart), (free(), left)
            else:
                with pytest.raises(S.StraitError) as e:
                    ctx.load(blob, max_batch=2, n_instances=1)
                assert e.value.status == S.E_NOMEM
    finally:
        filler.clear()
        torch.cuda.empty_cache()
    m = ctx.load(blob, max_batch=2, n_instances=1)
    try:
        assert np.array_equal(m.infer(x, vl)[0]["hidden"], folded)
    finally:
        m.free()


@pytest.mark.parametrize("hw,batch,fc", [(32, 5, 64), (64, 3, 256)])
def test_vgg19(ctx, hw, batch, fc):
    md = synth.vgg19(synth.SEEDS[synth.ARCH_VGG19], hw=hw, classes=100, fc=fc)
    x = synth.default_image_batch(md, batch, synth.SEEDS[synth.ARCH_VGG19] + batch)
    m, out, ref = run_cnn(ctx, md, x, omodels.vgg19_forward, ctx.S.PRIO_LOW, f"VGG-19 {hw}px b{batch}")
    m.free()


def test_vgg19_layers(ctx):
    """Every layer's activation against the oracle's: pooling positions, the flattening order into fc1."""
    md = synth.vgg19(4, hw=64, classes=10, fc=64)
    x = synth.default_image_batch(md, 2, 9)
    m = ctx.load(synth.pack(md), max_batch=2, n_instances=1)
    ref = omodels.vgg19_forward(md.tensors, x, keep=True)
    m.copy_in(0, ctx.S.PRIO_LOW, x)
    m.run(0, ctx.S.PRIO_LOW, 2)
    m.sync(0, ctx.S.PRIO_LOW)
    names = {li.name.decode(): i for i, li in enumerate(m.layers())}
    checked = 0
    for lname, act in ref.trace.acts.items():
        if lname not in names or lname == "fc":
            continue
        got = m.read_activation(0, names[lname], 2).astype(np.float64).reshape(act.shape)
        check_kernel(got, act, f"layer {lname}", rel=2.0 ** -8, abs_rel=1e-2)
        checked += 1
    assert checked == 16 + 5 + 2
    m.free()


def run_vit(ctx, md, x, what):
    m = ctx.load(synth.pack(md), max_batch=x.shape[0], n_instances=1)
    out, rec = m.infer(x, prio=ctx.S.PRIO_HIGH)
    ref = omodels.vit_forward(md.tensors, x, md.hyper, keep=True)
    err, scale, ties = check_logits(out["logits"], ref.logits, out["top1"], what)
    assert np.abs(out["probs"] - ref.probs).max() <= 2e-2
    print(f"{what}: max|err| {err:.3e} of scale {scale:.3e} ({err / scale:.2e}), ties {ties}, kernels {rec.kernel_ms:.3f} ms")
    return m, out, ref


@pytest.mark.parametrize("hw,batch,kw", [(48, 3, dict(layers=2, hidden=128, heads=2, ffn=256)),     # 10 tokens
                                         (96, 2, dict(layers=2, hidden=128, heads=2, ffn=256)),     # 37 tokens
                                         (224, 2, dict(layers=2, hidden=192, heads=3, ffn=384))])   # 197 tokens
def test_vit(ctx, hw, batch, kw):
    md = synth.vit(synth.SEEDS[synth.ARCH_VIT], hw=hw, classes=100, **kw)
    x = synth.default_image_batch(md, batch, synth.SEEDS[synth.ARCH_VIT] + batch)
    m, out, ref = run_vit(ctx, md, x, f"ViT {hw}px b{batch}")
    # every block's output (the residual stream) against the oracle's
    names = {li.name.decode(): i for i, li in enumerate(m.layers())}
    m.copy_in(0, ctx.S.PRIO_LOW, x)
    m.run(0, ctx.S.PRIO_LOW, batch)
    m.sync(0, ctx.S.PRIO_LOW)
    checked = 0
    for lname in ("patch", "tokens", "l0.qkv", "l0.attn", "l0.o", "l0.ffn1", "l0.ffn2", "l1.o", "l1.ffn2", "ln"):
        act = ref.trace.acts[lname]
        got = m.read_activation(0, names[lname], batch).astype(np.float64).reshape(act.shape)
        check_kernel(got, act, f"layer {lname}", rel=2.0 ** -8, abs_rel=1e-2)
        checked += 1
    assert checked == 10
    m.free()


def test_submit_errors_and_pool(ctx):
    S = ctx.S
    md = synth.tiny_cnn(1)
    m = ctx.load(synth.pack(md), max_batch=2, n_instances=2)
    x = synth.default_image_batch(md, 2, 1)
    outs = [m.new_output(2) for _ in range(3)]
    t0 = m.submit(S.PRIO_HIGH, x, None, outs[0])
    t1 = m.submit(S.PRIO_LOW, x, None, outs[1])
    assert m.try_submit(S.PRIO_LOW, x, None, outs[2]) is None            # both instances taken: E_BUSY, never blocks
    with pytest.raises(S.StraitError) as e:
        m.free()
    assert e.value.status == S.E_BUSY
    r0, r1 = m.wait(t0), m.wait(t1)
    assert {r0.instance, r1.instance} == {0, 1} and r0.priority == S.PRIO_HIGH and r1.priority == S.PRIO_LOW
    assert np.array_equal(outs[0], outs[1])                              # same input, either priority: same bits
    with pytest.raises(S.StraitError) as e:
        m.submit(S.PRIO_HIGH, synth.default_image_batch(md, 3, 1), None, m.new_output(2))
    assert e.value.status == S.E_BATCH
    m.free()
    with pytest.raises(S.StraitError) as e:
        ctx.load(b"STRX" + bytes(100), 1, 1)
    assert e.value.status == S.E_FORMAT


@pytest.mark.parametrize("arch,hw,classes,batch", [("tiny_cnn", 32, 10, 4), ("tiny_cnn", 20, 2, 3), ("tiny_cnn", 33, 256, 31), ("tiny_cnn", 32, 7, 300),   # pooling, product, softmax
                                                   ("tiny_cnn", 32, 257, 2), ("tiny_cnn", 32, 1023, 5), ("mobilenet_v2", 64, 1000, 32), ("mobilenet_v2", 64, 1024, 3),  # softmax
                                                   ("mobilenet_v2", 64, 1000, 33), ("tiny_cnn", 32, 1025, 2)])                                 # launches of their own
def test_classifier_results_that_leave_in_the_launch_that_computes_them(ctx, arch, hw, classes, batch):
    """Every form of the classifier's end, eager and replayed: the oracle's result, the same bytes on the device and from replays, and what the layers
    by themselves give (fp32 sums of up to 1024 terms in another order: 1024 * 2^-24 of the largest probability; a pooled feature may round the other
    way, 2^-10 of it)."""
    S = ctx.S
    md = getattr(synth, arch)(7, hw=hw, classes=classes)
    x = synth.default_image_batch(md, batch, 11)
    ref = (omodels.tiny_cnn_forward if arch == "tiny_cnn" else omodels.mobilenet_v2_forward)(md.tensors, x, keep=True)
    m = ctx.load(synth.pack(md), max_batch=batch, n_instances=1)
    try:
        m.copy_in(0, S.PRIO_LOW, x)
        m.run(0, S.PRIO_LOW, batch)
        apart = m.decode(m.copy_out(0, S.PRIO_LOW, batch), batch)
        first = None
        for graphs in (False, True, True, True, True):
            ctx.set_graphs(graphs)
            out = m.new_output(batch)
            rec = m.wait(m.submit(S.PRIO_HIGH, x, None, out))
            assert rec.kernel_ms > 0 and rec.d2h_ms > 0 and rec.total_ms >= rec.kernel_ms
            if first is None:
                first = out
            assert np.array_equal(first, out), "a pass differs from the first"
            assert np.array_equal(m.copy_out(0, S.PRIO_HIGH, batch).view(np.uint8), out.view(np.uint8)), "the device's copy differs"
        got = m.decode(first, batch)
        check_logits(got["logits"], ref.logits, got["top1"], f"{arch} {classes} classes b{batch}")
        assert np.abs(got["probs"] - ref.probs).max() <= 2e-2 and np.abs(got["probs"].sum(-1) - 1).max() < 1e-4
        assert np.array_equal(got["top1"], got["logits"].argmax(-1))
        if arch == "tiny_cnn" and classes <= 256:
            assert np.abs(got["logits"] - apart["logits"]).max() <= 2.0 ** -10 * np.abs(md.tensors["fc.w"].astype(np.float64)).sum(1).max() * ref.trace.acts["gap"].max()
        else:
            assert np.array_equal(got["logits"], apart["logits"]) and np.array_equal(got["top1"], apart["top1"])
            assert np.abs(got["probs"] - apart["probs"]).max() <= 2 * 1024 * 2.0 ** -24 * apart["probs"].max()
    finally:
        ctx.set_graphs(False)
        m.free()


@pytest.mark.parametrize("arch,hw,classes,batch", [("tiny_cnn", 33, 256, 31), ("mobilenet_v2", 64, 1000, 4)])
def test_the_layer_by_layer_plan_ends_in_its_own_launches(ctx, arch, hw, classes, batch):
    """set_pair_fusion(0): a submitted batch, eager, replayed or in segments, is what its layers by themselves give, to the last bit."""
    S = ctx.S
    md = getattr(synth, arch)(7, hw=hw, classes=classes)
    x = synth.default_image_batch(md, batch, 11)
    m = ctx.load(synth.pack(md), max_batch=batch, n_instances=1)
    ctx.set_pair_fusion(0)
    try:
        m.copy_in(0, S.PRIO_LOW, x)
        m.run(0, S.PRIO_LOW, batch)
        apart = m.copy_out(0, S.PRIO_LOW, batch)
        for graphs, segment in ((False, 0), (True, 0), (True, 0), (True, 0), (False, 2)):
            ctx.set_graphs(graphs)
            ctx.set_lp_yield(segment)
            out = m.new_output(batch)
            m.wait(m.submit(S.PRIO_LOW, x, None, out))
            assert np.array_equal(out.view(np.uint8), apart.view(np.uint8)), (graphs, segment)
    finally:
        ctx.set_graphs(False)
        ctx.set_lp_yield(0)
        ctx.set_pair_fusion(40000)
        m.free()


def test_more_rows_than_the_gpu_takes_at_a_time_end_in_launches_of_their_own(ctx):
    """1024 rows take their results along in the launch that computes them, 1025 do not: the bytes that the layers by themselves give, and in both cases the
    same ones pass after pass and the oracle's (rows are counted in groups of 32, the last one whole or a single row)."""
    S = ctx.S
    md = synth.tiny_cnn(7, hw=32, classes=10)
    x = synth.default_image_batch(md, 1025, 11)
    ref = omodels.tiny_cnn_forward(md.tensors, x)
    m = ctx.load(synth.pack(md), max_batch=1025, n_instances=1)
    try:
        for b in (1025, 1024, 993, 33, 32):
            m.copy_in(0, S.PRIO_LOW, x[:b])
            m.run(0, S.PRIO_LOW, b)
            apart = m.copy_out(0, S.PRIO_LOW, b)
            for k in range(4):
                out = m.new_output(b)
                m.wait(m.submit(S.PRIO_LOW, x[:b], None, out))
                if k == 0:
                    first = out
                assert np.array_equal(out.view(np.uint8), first.view(np.uint8)), (b, k)
            assert np.array_equal(out.view(np.uint8), apart.view(np.uint8)) == (b == 1025), b
            got = m.decode(out, b)
            check_logits(got["logits"], ref.logits[:b], got["top1"], f"{b} rows")
    finally:
        m.free()


@pytest.mark.parametrize("h,w,classes,batch", [(1, 1, 4, 1), (2, 3, 10, 5), (7, 40, 255, 3), (31, 33, 12, 33), (32, 32, 256, 2), (45, 46, 10, 2), (48, 47, 10, 2)])
def test_a_small_network_in_one_launch(ctx, h, w, classes, batch):
    """Images of one pixel, odd and oblong ones, about the largest and one too large, the largest head: the oracle's result, with infinities and a NaN among the pixels too, where it has to be
    infinite, zero or no number in the same places as layer by layer."""
    S = ctx.S
    md = synth.tiny_cnn(7, hw=32, classes=classes)
    md = synth.ModelData(md.arch, (h, w, 3, classes), md.tensors)
    x = np.random.default_rng(3).random((batch, h, w, 3), dtype=np.float32).astype(np.float16)
    ref = omodels.tiny_cnn_forward(md.tensors, x)
    m = ctx.load(synth.pack(md), max_batch=batch, n_instances=1)
    try:
        got, _ = m.infer(x)
        check_logits(got["logits"], ref.logits, got["top1"], f"tiny CNN {h} x {w}, {classes} classes, b{batch}")
        assert np.abs(got["probs"] - ref.probs).max() <= 2e-2
        x[0, h // 2, w // 2] = (np.inf, 0, 0)
        x[batch - 1, h - 1, 0] = (0, -np.inf, np.nan)
        odd = []
        for fusion in (40000, 0):
            ctx.set_pair_fusion(fusion)
            odd.append(m.infer(x)[0])
        assert np.array_equal(np.isnan(odd[0]["logits"]), np.isnan(odd[1]["logits"])) and np.array_equal(np.isinf(odd[0]["logits"]), np.isinf(odd[1]["logits"]))
        fine = np.isfinite(odd[1]["logits"])
        assert np.allclose(odd[0]["logits"][fine], odd[1]["logits"][fine], rtol=0, atol=2e-2 * max(1.0, np.abs(odd[1]["logits"][fine]).max(initial=0)))
    finally:
        ctx.set_pair_fusion(40000)
        m.free()


@pytest.mark.parametrize("hw,batch", [(8, 1521), (10, 1058)])
def test_many_small_images_are_packed_for_the_first_layer(ctx, hw, batch):
    """Images that leave most of the direct first layer's tiles empty, one more of them than it takes: the layer-by-layer plan's bytes."""
    S = ctx.S
    md = synth.tiny_cnn(7, hw=hw, classes=10)
    x = synth.default_image_batch(md, batch, 11)
    m = ctx.load(synth.pack(md), max_batch=batch, n_instances=1)
    try:
        got = []
        for fusion in (40000, 0):
            ctx.set_pair_fusion(fusion)
            out = m.new_output(batch)
            m.wait(m.submit(S.PRIO_LOW, x, None, out))
            got.append(out.view(np.uint8).copy())
        assert np.array_equal(*got)
    finally:
        ctx.set_pair_fusion(40000)
        m.free()


def test_kernel_time_covers_every_row(ctx):
    """1024 rows whose pooling, product and softmax share a launch with the result's way out: the computation does not end with the first row.  What is left
    then is the way of the rows' 84 bytes to the host, 4.5 us in a median of eight (12 with the first row's end and one counter for all rows)."""
    S = ctx.S
    md = synth.tiny_cnn(7, hw=32, classes=10)
    x = np.random.default_rng(1).random((1024, 32, 32, 3), dtype=np.float32).astype(np.float16)
    m = ctx.load(synth.pack(md), max_batch=1024, n_instances=1)
    try:
        out = m.new_output(1024)
        recs = [m.wait(m.submit(S.PRIO_HIGH, x, None, out)) for _ in range(9)][1:]
        assert 0 < np.median([r.d2h_ms for r in recs]) < 0.008
        assert all(r.kernel_ms > 0 and r.total_ms >= r.kernel_ms + r.d2h_ms for r in recs)
    finally:
        m.free()


def test_small_results_on_alternating_streams(ctx):
    """One instance, its batches by turns on two compute streams and of two sizes, so that one batch's probabilities lie where the next one's logits do:
    each result, and the device's copy read through the other stream as soon as the host has the result, is what it was the first time."""
    S = ctx.S
    md = synth.tiny_cnn(7, hw=32, classes=256)
    m = ctx.load(synth.pack(md), max_batch=31, n_instances=1)
    jobs = [(b, synth.default_image_batch(md, b, 11 + b), prio, other) for b, prio, other in
            ((3, S.PRIO_HIGH, S.PRIO_LOW), (31, S.PRIO_LOW, S.PRIO_HIGH), (1, S.PRIO_HIGH, S.PRIO_LOW), (30, S.PRIO_LOW, S.PRIO_HIGH))]
    first = {}
    try:
        for k in range(50):
            for b, x, prio, other in jobs:
                out = m.new_output(b)
                m.wait(m.submit(prio, x, None, out))
                if k % 5 == 0:                             # otherwise the next batch follows at once
                    assert np.array_equal(m.copy_out(0, other, b).view(np.uint8), out.view(np.uint8)), f"pass {k}, batch {b}: the device's copy differs"
                assert np.array_equal(first.setdefault(b, out), out), f"pass {k}, batch {b}: differs from the first"
    finally:
        m.free()


@pytest.mark.parametrize("arch,batch", [("resnet50", 3), ("mobilenet_v2", 4), ("encoder", 2)])
def test_graph_replay_equals_kernel_by_kernel(ctx, arch, batch):
    """The captured-graph path replays the very same launches: every replay, on fresh inputs and with
    kernel-by-kernel passes and synchronisations in between, must equal the eager result bit for bit."""
    S = ctx.S
    if arch == "encoder":
        md = synth.encoder(5, layers=2, hidden=128, heads=2, ffn=256, seq=64)
    else:
        md = getattr(synth, arch)(5, hw=64)
    m = ctx.load(synth.pack(md), max_batch=batch, n_instances=2)
    try:
        for rep in range(5):                      # first use of a key runs eagerly, the second captures, later ones replay
            if arch == "encoder":
                x, vl = synth.token_batch(md, batch, 50 + rep)
            else:
                x, vl = synth.default_image_batch(md, batch, 50 + rep), None
            for prio in (S.PRIO_HIGH, S.PRIO_LOW):
                ctx.set_graphs(False)
                eager = m.new_output(batch)
                m.wait(m.submit(prio, x, vl, eager))
                ctx.set_graphs(True)
                replay = m.new_output(batch)
                rec = m.wait(m.submit(prio, x, vl, replay))
                assert np.array_equal(eager.view(np.uint8), replay.view(np.uint8)), (arch, rep, prio)
                assert rec.kernel_ms > 0
    finally:
        ctx.set_graphs(False)
        m.free()


def test_graphs_recorded_while_an_earlier_batch_is_awaited(ctx):
    """A batch of tens of milliseconds is being waited for, and its stream asked every few milliseconds whether it is well, while the batches
    behind it record their graphs on the same stream, one after the other: neither disturbs the other."""
    S = ctx.S
    slow_md = synth.encoder(3, layers=6, hidden=768, heads=12, ffn=3072, seq=256)
    slow_b, quick_n = 512, 48
    x8, vl8 = synth.token_batch(slow_md, 8, 1, min_len=32)
    rows = np.arange(slow_b) % 8
    x, vl = x8[rows], vl8[rows]
    md = synth.resnet50(9, hw=64)
    xq = synth.default_image_batch(md, 1, 3)
    slow = ctx.load(synth.pack(slow_md), max_batch=slow_b, n_instances=2)
    quick = ctx.load(synth.pack(md), max_batch=1, n_instances=quick_n)
    try:
        ctx.set_graphs(True)
        for i in range(quick_n):                  # the first use of an instance runs without a graph
            buf = quick.staging(i, 1)
            buf[:] = xq
            ref, _ = quick.infer(buf, prio=S.PRIO_LOW)
        out = [slow.new_output(slow_b) for _ in range(2)]
        outq = [quick.new_output(1) for _ in range(quick_n)]
        tickets = [slow.submit(S.PRIO_LOW, x, vl, o) for o in out]
        tq = [quick.submit(S.PRIO_LOW, quick.staging(i, 1), None, outq[i]) for i in range(quick_n)]
        for t in tickets:
            slow.wait(t)
        for t in tq:
            quick.wait(t)
        assert np.array_equal(out[0], out[1])
        for o in outq:
            assert np.array_equal(quick.decode(o, 1)["logits"], ref["logits"])
    finally:
        ctx.set_graphs(False)
        slow.free()
        quick.free()


def test_small_batch_split_reduction_is_reproducible(ctx):
    """Small batches split long reductions over several workgroups per tile; the partial results are summed
    in a fixed order, so repeated runs must agree bit for bit, at either priority."""
    S = ctx.S
    md = synth.resnet50(9, hw=64)
    x = synth.default_image_batch(md, 2, 3)
    m = ctx.load(synth.pack(md), max_batch=2, n_instances=2)
    try:
        outs = []
        for rep in range(6):
            out = m.new_output(2)
            m.wait(m.submit(S.PRIO_HIGH if rep % 2 else S.PRIO_LOW, x, None, out))
            outs.append(out.copy())
        for o in outs[1:]:
            assert np.array_equal(o.view(np.uint8), outs[0].view(np.uint8))
        ref = omodels.resnet50_forward(md.tensors, x)
        check_logits(m.decode(outs[0], 2)["logits"], ref.logits, m.decode(outs[0], 2)["top1"], "ResNet-50 64px b2 (split reductions)")
    finally:
        m.free()


def test_input_copy_by_kernel_and_by_copy_engine_give_the_same_result(ctx):
    """Inputs up to a settable size go in by a copy kernel, larger ones by hipMemcpyAsync: same bytes on the device
    either way, so outputs are identical bit for bit."""
    md = synth.resnet50(4, hw=64)
    m = ctx.load(synth.pack(md), max_batch=4, n_instances=1)
    try:
        x = synth.default_image_batch(md, 4, 3)
        outs = []
        for limit in (0, 8 << 20):
            ctx.set_h2d_kernel_limit(limit)
            out, rec = m.infer(x)
            assert rec.h2d_ms > 0
            outs.append(out)
        assert np.array_equal(outs[0]["logits"], outs[1]["logits"]) and np.array_equal(outs[0]["top1"], outs[1]["top1"])
    finally:
        ctx.set_h2d_kernel_limit(8 << 20)
        m.free()


@pytest.mark.parametrize("batch", [1, 2, 6, 33])
def test_transfers_in_pieces_bring_every_byte(ctx, batch):
    """128 KB in and 128 KB + 4 B out per sequence: results of one part, of whole chunks and a few bytes, and one that leaves on a copy
    stream; inputs of one and of several pieces; two batches in flight, so one input goes in on the compute stream and one
    beside it.  Same kernels as the copy-call sub-steps: identical bit for bit."""
    S = ctx.S
    md = synth.encoder(3, layers=1, hidden=256, heads=4, ffn=256, seq=256)
    m = ctx.load(synth.pack(md), max_batch=batch, n_instances=2)
    try:
        xs = [synth.token_batch(md, batch, seed, min_len=32) for seed in (1, 2)]
        refs = []
        for x, vl in xs:
            m.copy_in(0, S.PRIO_LOW, x, vl)
            m.run(0, S.PRIO_LOW, batch)
            refs.append(m.copy_out(0, S.PRIO_LOW, batch))
        for _ in range(3):
            outs = [m.new_output(batch) for _ in xs]
            tickets = [m.submit(S.PRIO_LOW, x, vl, o) for (x, vl), o in zip(xs, outs)]
            for t in tickets:
                rec = m.wait(t)
                assert rec.h2d_ms > 0 and rec.kernel_ms > 0 and rec.d2h_ms > 0
            assert all(np.array_equal(o, r) for o, r in zip(outs, refs))
    finally:
        m.free()


def test_one_instance_handed_from_stream_to_stream(ctx):
    """Results of several chunks, one instance, the priority and so the compute stream changing from batch to batch without a pause:
    the counters that tell the last part of a chunk are the instance's and have to be back at zero for the next stream."""
    S = ctx.S
    md = synth.encoder(3, layers=1, hidden=256, heads=4, ffn=256, seq=256)
    m = ctx.load(synth.pack(md), max_batch=33, n_instances=1)
    try:
        want = {}
        for i in range(120):
            batch = (33, 6, 16)[i % 3]                    # 4.3 MB: leaves on a copy stream
            x, vl = synth.token_batch(md, batch, batch, min_len=32) if batch not in want else want[batch][0]
            out = m.new_output(batch)
            m.wait(m.submit((S.PRIO_HIGH, S.PRIO_LOW)[i & 1], x, vl, out))
            ref = want.setdefault(batch, ((x, vl), out))[1]
            assert np.array_equal(out, ref), i
    finally:
        m.free()


def test_large_inputs_in_pieces_from_two_threads(ctx):
    """19 MB in ordinary memory by the copy engine, in pieces, from two threads and through one and two copy streams at once: whole,
    in several pieces, or the rest in one after another batch's came between; always every byte."""
    import threading
    S = ctx.S
    md = synth.tiny_cnn(synth.SEEDS[synth.ARCH_TINY_CNN], hw=224)
    for n_copy in (1, 2):
        c = S.Context(device=0, n_hp=1, n_lp=1, n_copy=n_copy)
        m = c.load(synth.pack(md), max_batch=64, n_instances=2)
        try:
            xs = [synth.default_image_batch(md, 64, i) for i in range(2)]
            want = [m.infer(x)[0]["logits"].copy() for x in xs]
            bad = []

            def client(i):
                for _ in range(10):
                    out, rec = m.infer(xs[i], prio=(S.PRIO_HIGH, S.PRIO_LOW)[i])
                    if not np.array_equal(out["logits"], want[i]) or not 0 < rec.h2d_ms <= rec.total_ms:
                        bad.append((i, rec.h2d_ms, rec.total_ms))

            threads = [threading.Thread(target=client, args=(i,)) for i in range(2)]
            for t in threads:
                t.start()
            for t in threads:
                t.join()
            assert not bad
        finally:
            m.free()
            c.close()


def test_result_of_more_than_a_gibibyte(ctx):
    """2900 sequences of 393 KB: more 256 KB chunks than there are flags, so the chunks are larger.  Every row is the answer to one of
    eight sequences; a product's sums do not depend on the row, so equal sequences give equal rows."""
    S = ctx.S
    md = synth.encoder(3, layers=1, hidden=768, heads=12, ffn=256, seq=256)
    batch = 2900
    x8, vl8 = synth.token_batch(md, 8, 1, min_len=32)
    rows = np.arange(batch) % 8
    m = ctx.load(synth.pack(md), max_batch=batch, n_instances=1)
    try:
        out, _ = m.infer(x8[rows], vl8[rows], prio=S.PRIO_LOW)
        first = out["hidden"][:8].copy()
        small, _ = m.infer(x8, vl8, prio=S.PRIO_LOW)
        # fp16 results of 8 and of 2900 rows may come from kernels that add in another order
        assert np.abs(first.astype(np.float32) - small["hidden"].astype(np.float32)).max() <= 2e-2 * np.abs(small["hidden"]).max()
        for at in range(0, batch, 8):
            n = min(8, batch - at)
            assert np.array_equal(out["hidden"][at:at + n], first[:n]), at
            assert np.array_equal(out["top1"][at:at + n], out["top1"][:n]), at
    finally:
        m.free()


def test_submit_from_the_staging_buffer_makes_no_host_copy_and_gives_the_same_result(ctx):
    S = ctx.S
    md = synth.resnet50(4, hw=64)
    x = synth.default_image_batch(md, 3, 5)
    m = ctx.load(synth.pack(md), max_batch=4, n_instances=2)
    try:
        ref = m.new_output(3)
        m.wait(m.submit(S.PRIO_LOW, x, None, ref))
        st = m.staging(1, 3)                        # instance 1's pinned input buffer
        st[:] = x
        out = m.new_output(3)
        rec = m.wait(m.submit(S.PRIO_HIGH, st, None, out))
        assert rec.instance == 1 and np.array_equal(out, ref)
        t = m.submit(S.PRIO_HIGH, st, None, out)    # the same buffer again while its batch is in flight: refused, not queued
        with pytest.raises(S.StraitError) as e:
            m.submit(S.PRIO_HIGH, st, None, m.new_output(3))
        assert e.value.status == S.E_BUSY
        m.wait(t)
    finally:
        m.free()


@pytest.mark.parametrize("arch,kw,batch", [("mobilenet_v2", dict(hw=96), 171),                                      # 43, 86 and 42 images
                                           ("mobilenet_v2", dict(hw=96), 700),                                      # eight full parts and one of a half
                                           ("vgg19", dict(hw=64, classes=50, fc=64), 389),
                                           ("vit", dict(hw=96, classes=100, layers=2, hidden=128, heads=2, ffn=256), 171),
                                           ("encoder", dict(layers=3, hidden=128, heads=2, ffn=256, seq=40), 1001)])
def test_a_large_batch_begun_while_its_input_is_on_the_way(ctx, arch, kw, batch):
    """A staged input of 9 MB and more: the first layers of each part run while the next is on the link (the record's phases overlap).  Every sample's result is that of the same batch
    computed whole, to within what its layers' roundings to fp16 differ by where a part's products sum in another order."""
    S = ctx.S
    md = getattr(synth, arch)(21, **kw)
    x, vl = synth.token_batch(md, batch, 8) if arch == "encoder" else (synth.default_image_batch(md, batch, 8), None)
    m = ctx.load(synth.pack(md), max_batch=batch, n_instances=1)
    try:
        whole, parts = m.new_output(batch), m.new_output(batch)
        m.wait(m.submit(S.PRIO_LOW, x, vl, whole))                        # ordinary memory: in one go
        st = m.staging(0, batch)
        st[:] = x
        want = m.decode(whole, batch)
        key = "hidden" if arch == "encoder" else "logits"
        want = want[key].astype(np.float64).copy()
        for prio in (S.PRIO_HIGH, S.PRIO_LOW, S.PRIO_HIGH):
            parts[:] = 0
            rec = m.wait(m.submit(prio, st, vl, parts))
            got = m.decode(parts, batch)[key].astype(np.float64)
            if arch == "encoder":
                for i in range(batch):
                    check_kernel(got[i, :vl[i]], want[i, :vl[i]], f"sequence {i}", rel=2.0 ** -8, abs_rel=1e-2)
            else:
                check_kernel(got, want, f"{arch} b{batch}", rel=2.0 ** -8, abs_rel=1e-2)
            if arch != "encoder":                     # (whose large output starts when the host has seen its kernels done, which no phase holds)
                assert rec.h2d_ms + rec.kernel_ms + rec.d2h_ms > rec.total_ms, (rec.h2d_ms, rec.kernel_ms, rec.d2h_ms, rec.total_ms)
    finally:
        m.free()


@pytest.mark.parametrize("arch,kw,batch", [("vit", dict(hw=96, classes=100, layers=2, hidden=128, heads=2, ffn=256), 171),        # a part's products would split their reductions
                                           ("vit", dict(hw=96, classes=100, layers=2, hidden=128, heads=2, ffn=256), 613),
                                           ("vit", dict(hw=224, classes=100, layers=2), 45),
                                           ("encoder", dict(layers=3, hidden=128, heads=2, ffn=256, seq=40), 1001),
                                           ("encoder", dict(layers=2, hidden=768, heads=12, ffn=3072, seq=128), 50),
                                           ("mobilenet_v2", dict(hw=96), 171), ("mobilenet_v2", dict(hw=224), 64),
                                           ("vgg19", dict(hw=64, classes=50, fc=64), 389),
                                           # images' bytes and tokens' statistics that are no multiples of 16
                                           ("mobilenet_v2", dict(hw=250), 64), ("mobilenet_v2", dict(hw=226), 57), ("tiny_cnn", dict(hw=30), 1801),
                                           ("encoder", dict(layers=2, hidden=64, heads=1, ffn=256, seq=37), 2001),
                                           ("vit", dict(hw=224, classes=100, layers=2, hidden=192, heads=3, ffn=768), 33)])
def test_a_batch_in_parts_gives_the_bytes_of_the_whole(ctx, arch, kw, batch):
    """Whether a staged batch of 9 MB and more goes in parts depends on what else is on its way.  Its result does not: parts take kernels that add in the whole batch's order."""
    S = ctx.S
    md = getattr(synth, arch)(22, **kw)
    x, vl = synth.token_batch(md, batch, 9) if arch == "encoder" else (synth.default_image_batch(md, batch, 9), None)
    m = ctx.load(synth.pack(md), max_batch=batch, n_instances=1)
    try:
        whole, parts = m.new_output(batch), m.new_output(batch)
        m.wait(m.submit(S.PRIO_LOW, x, vl, whole))                        # ordinary memory: in one go
        st = m.staging(0, batch)
        st[:] = x
        for prio in (S.PRIO_HIGH, S.PRIO_LOW):
            parts[:] = 0
            m.wait(m.submit(prio, st, vl, parts))
            assert np.array_equal(parts, whole), (arch, batch, prio)
    finally:
        m.free()


def test_other_threads_submit_while_a_batch_goes_in_parts(ctx):
    """Two threads with a large staged batch each and one with small batches share a compute stream, a fourth has the other level's: batches are enqueued between the parts of another one.
    Every result is that of the batch by itself."""
    import threading
    S = ctx.S
    big, small = synth.mobilenet_v2(23), synth.tiny_cnn(23, hw=64)
    mb, ms = ctx.load(synth.pack(big), max_batch=64, n_instances=2), ctx.load(synth.pack(small), max_batch=8, n_instances=2)
    try:
        xb = [synth.default_image_batch(big, n, 30 + n) for n in (64, 50)]
        xs = [synth.default_image_batch(small, 8, 40 + i) for i in range(2)]
        want_b = [mb.infer(x, prio=S.PRIO_LOW)[0]["logits"].copy() for x in xb]
        want_s = [ms.infer(x, prio=S.PRIO_LOW)[0]["logits"].copy() for x in xs]
        staged = [mb.staging(i, len(xb[i])) for i in range(2)] + [ms.staging(i, 8) for i in range(2)]
        for st, x in zip(staged, xb + xs):
            st[:] = x
        bad, gate = [], threading.Barrier(4)

        def work(model, st, prio, want, times):
            out = model.new_output(len(st))
            gate.wait()
            for k in range(times):
                rec = model.wait(model.submit(prio, st, None, out))
                if not np.array_equal(model.decode(out, len(st))["logits"], want) or not rec.kernel_ms <= rec.total_ms:
                    bad.append((model.arch, len(st), prio, k, rec.kernel_ms, rec.total_ms))

        jobs = [(mb, staged[0], S.PRIO_LOW, want_b[0], 25), (mb, staged[1], S.PRIO_LOW, want_b[1], 25), (ms, staged[2], S.PRIO_LOW, want_s[0], 200), (ms, staged[3], S.PRIO_HIGH, want_s[1], 200)]
        th = [threading.Thread(target=work, args=j) for j in jobs]
        for t in th:
            t.start()
        for t in th:
            t.join()
        assert not bad, bad[:5]
    finally:
        mb.free()
        ms.free()
