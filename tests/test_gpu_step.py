"""GPU parity of cnnk_train_step against the oracle walker: loss, every activation, every
activation gradient, every parameter gradient, updated weights and momentum, labels/argmax."""
import numpy as np
import pytest
import torch

import workloads as WL
from util import JITTER_REL, JITTER_SEEDS, SCALE_TO_EXACT, SCALE_TO_MEMBER, TOL, ensemble_bound, host, max_rel_err

pytestmark = pytest.mark.gpu

import oracle  # noqa: E402


def run_both(net, config_id, lr=0.1, momentum=0.9, wd=0.0, steps=1, **gen):
    """Runs the HIP step and the oracle walker(s) on the same seeded inputs.  For the bf16 mode the
    oracle is walked in pure float64 (key None) and as an ensemble of equally legal bf16-storage
    walks: the plain one (key "bf16") and one per seed of JITTER_SEEDS (key ("bf16", seed)) whose
    roundings are decided on values perturbed by an fp32-accumulation-sized amount (see
    oracle/step.py)."""
    from paper_2503_23186_amd import StepRunner
    inp = WL.make_inputs(net, config_id, **gen)
    runner = StepRunner(net.layers, net.slots, [p["shape"] for p in net.params], net.dtype)
    runner.load(inp["x"], inp["labels"], inp["params"], inp["mom"])
    modes = [None]
    if net.dtype == "bf16":
        modes += ["bf16"] + [("bf16", s) for s in JITTER_SEEDS]
    outs = {}
    state = {m: (inp["params"], inp["mom"]) for m in modes}
    for k in range(steps):
        runner.step(lr, momentum, wd)
        for m in modes:
            storage = None if m is None else "bf16"
            jitter = (1000 * m[1] + k, JITTER_REL) if isinstance(m, tuple) else None
            outs[m] = oracle.train_step(net, inp["x"], inp["labels"], state[m][0], state[m][1], lr, momentum, wd,
                                        storage=storage, jitter=jitter)
            state[m] = (outs[m]["params"], outs[m]["mom"])
    torch.cuda.synchronize()
    return inp, runner, outs


def l2_rel_err(got, ref):
    return float(np.linalg.norm((got - ref).ravel()) / max(np.linalg.norm(ref.ravel()), 1e-30))


def runner_tensors(runner, like):
    """The HIP step's tensors as host float64 arrays, in the layout of an oracle result."""
    return dict(loss=runner.loss.item(),
                acts={s: host(runner.act[s]).reshape(a.shape) for s, a in like["acts"].items()},
                dacts={s: host(runner.dact[s]).reshape(g.shape) for s, g in like["dacts"].items()},
                grads=[host(runner.grad[k]).reshape(g.shape) for k, g in enumerate(like["grads"])],
                params=[host(runner.param[k]).reshape(g.shape) for k, g in enumerate(like["params"])],
                mom=[host(runner.mom[k]).reshape(g.shape) for k, g in enumerate(like["mom"])],
                probs=host(runner.probs))


def errors(got, out):
    """Per tensor class: worst max-norm error (max|got-ref| / max|ref|) and worst L2 relative error
    of `got` against `out` (both in the layout of an oracle result)."""
    e = {}

    def upd(kind, a, b):
        m, l = max_rel_err(a, b), l2_rel_err(a, b)
        pm, pl = e.get(kind, (0.0, 0.0))
        e[kind] = (max(pm, m), max(pl, l))

    upd("loss", np.array([got["loss"]]), np.array([out["loss"]]))
    for s, a in out["acts"].items():
        if s != 0:
            upd("act", got["acts"][s], a)
    for s, g in out["dacts"].items():
        upd("dact", got["dacts"][s], g)
    for k, g in enumerate(out["grads"]):
        upd("grad", got["grads"][k], g)
        upd("param", got["params"][k], out["params"][k])
        upd("mom", got["mom"][k], out["mom"][k])
    upd("probs", got["probs"], out["probs"])
    return e


def check_step(net, inp, runner, outs, tol):
    """fp32 mode: every tensor within `tol` (max-norm) of the float64 oracle.

    bf16 mode: a free-running bf16 step and the float64 walk decide ReLU masks and pool winners on
    values that differ by storage rounding, and at random initialisation the gradients are
    incoherent sums, so a fraction f of flipped decisions moves a gradient by about sqrt(f) of its
    norm whatever the implementation.  How far a correct bf16 implementation may lie from the
    float64 walk, and from another correct one, is measured on the oracle alone: an ensemble of
    bf16-storage walks that differ only in roundings an fp32 accumulation could decide either way.
    The HIP step has to be statistically indistinguishable from a member (oracle.ensemble: the
    members' mean figure, scaled for the factor of two to which the ensemble's noise amplitude
    models the implementation's, + 3 standard deviations of the members' own figures + `tol`) in
      (a) its L2 distance to the float64 walk, per tensor class,
      (b) its mean L2 distance to the members, against the members' pairwise distances,
      (c) for the forward quantities (activations, probabilities), which are not chaotic, also
          the max-norm distance to the float64 walk;
    the loss is within `tol` of the float64 loss outright.  The max-norm of a gradient is one
    worst element of a chaotic quantity and is graded where it is well posed: element-wise bf16
    parity of every layer on identical inputs (test_gpu_layers.py, test_gpu_fullsize.py)."""
    assert torch.equal(runner.labels.cpu(), torch.from_numpy(inp["labels"]))        # labels pass through
    for k in range(len(net.params)):
        if runner.param_lp[k] is not None:
            assert torch.equal(runner.param_lp[k], runner.param[k].to(torch.bfloat16))
    pure = outs[None]
    hip = runner_tensors(runner, pure)
    e = errors(hip, pure)
    print("\n%s [%s] b%d vs float64 oracle (max-norm/L2): %s"
          % (net.name, net.dtype, net.batch, {k: "%.1e/%.1e" % v for k, v in e.items()}))
    p = pure["probs"]
    top2 = np.sort(p, axis=1)[:, -2:]
    pred = runner.pred.cpu().numpy()
    if net.dtype == "f32":
        for kind, (m, _) in e.items():
            assert m <= tol, (kind, m)
        safe = (top2[:, 1] - top2[:, 0]) > 4 * tol * top2[:, 1]
    else:
        members = [outs["bf16"]] + [outs[("bf16", s)] for s in JITTER_SEEDS]
        to_pure = [errors(m, pure) for m in members]
        pairs = [errors(members[i], members[j]) for i in range(len(members)) for j in range(i)]
        to_members = [errors(hip, m) for m in members]
        assert e["loss"][0] <= tol, e["loss"]
        report = {}
        for kind in ("act", "dact", "grad", "param", "mom", "probs"):
            b_pure = ensemble_bound([t[kind][1] for t in to_pure], tol, SCALE_TO_EXACT)
            b_pair = ensemble_bound([t[kind][1] for t in pairs], tol, SCALE_TO_MEMBER)
            d_mem = float(np.mean([t[kind][1] for t in to_members]))
            report[kind] = "%.1e<=%.1e %.1e<=%.1e" % (e[kind][1], b_pure, d_mem, b_pair)
            assert e[kind][1] <= b_pure, (kind, "L2 distance to the float64 walk", e[kind][1], b_pure)
            assert d_mem <= b_pair, (kind, "mean L2 distance to the ensemble", d_mem, b_pair)
            if kind in ("act", "probs"):
                b_max = ensemble_bound([t[kind][0] for t in to_pure], tol, SCALE_TO_EXACT)
                assert e[kind][0] <= b_max, (kind, "max-norm distance to the float64 walk", e[kind][0], b_max)
        print("%s L2: to float64 <= ensemble bound, to members <= pairwise bound: %s" % (net.name, report))
        safe = (top2[:, 1] - top2[:, 0]) > 4 * max(tol, e["probs"][0]) * top2[:, 1]
    assert np.array_equal(pred[safe], pure["pred"][safe])                            # argmax: bit exact
    print("argmax compared on %d of %d samples" % (int(safe.sum()), len(safe)))


def test_config1_tiny_cnn_fp32():
    net = WL.build_config(1)
    inp, runner, out = run_both(net, 1)
    check_step(net, inp, runner, out, TOL["f32"])


def test_config1_three_steps_zero_initial_momentum():
    net = WL.build_config(1)
    inp, runner, out = run_both(net, 1, steps=3, zero_momentum=True)
    check_step(net, inp, runner, out, TOL["f32"])


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("name", ["mini_resnet", "mini_preact"])
def test_mini_nets(name, dtype):
    net = getattr(WL, name)(batch=6, dtype=dtype, size=8, widths=(16, 32))
    inp, runner, out = run_both(net, 60, perturb_bn=True, wd=5e-4)
    check_step(net, inp, runner, out, TOL[dtype])


def test_config2_vgg_bf16_batch16():
    net = WL.build_config(2, batch=16)
    inp, runner, out = run_both(net, 2)
    check_step(net, inp, runner, out, TOL["bf16"])


def test_config3_resnet18_bf16_batch8():
    net = WL.build_config(3, batch=8)
    inp, runner, out = run_both(net, 3)
    check_step(net, inp, runner, out, TOL["bf16"])


def test_config4_resnet50_bf16_batch4():
    net = WL.build_config(4, batch=4)
    inp, runner, out = run_both(net, 4)
    check_step(net, inp, runner, out, TOL["bf16"])


def test_config5_wrn_bf16_small():
    net = WL.wrn28_10(batch=4, widths=(32, 64, 128), per_group=2)
    inp, runner, out = run_both(net, 5)
    check_step(net, inp, runner, out, TOL["bf16"])


def test_fp32_resnet18_narrow():
    net = WL.resnet18(batch=4, dtype="f32", size=16, widths=(16, 32, 64, 128))
    inp, runner, out = run_both(net, 30)
    check_step(net, inp, runner, out, TOL["f32"])


def uses_second_stream(net):
    """Steps of little work leave it unused; 46 GFLOP of convolutions are enough whatever their weights."""
    return net.conv_flops()[1] > 46e9


def _two_stream_net():
    net = WL.mini_resnet(batch=64, dtype="bf16", size=32, widths=(64, 128))
    assert uses_second_stream(net)
    return net


@pytest.mark.parametrize("group", [1, 2])
def test_two_streams_match_one_stream(group):
    """The weight gradients forked onto a second stream give the results of the single-stream
    order over several consecutive steps (workspace halves and events reused).  The forked
    weight gradients split their pixel range over fewer workgroups, so the fp32 partial sums are
    grouped differently: equal up to fp32 rounding, and each mode is bit-reproducible.  Forked one by one and in pairs
    (tune key 17)."""
    net = _two_stream_net()
    inp = WL.make_inputs(net, 0)
    a, b, c = (_run_steps(net, inp, {17: group}, two_streams=two, steps=3) for two in (False, True, True))
    assert abs(a.loss.item() - b.loss.item()) <= 1e-5 * abs(a.loss.item())
    for k in range(len(net.params)):
        for name in ("grad", "param", "mom"):
            ta, tb, tc = (getattr(r, name)[k] for r in (a, b, c))
            assert torch.equal(tb, tc), "%s %d differs between two identical runs" % (name, k)
            scale = ta.abs().max().item() + 1e-30
            assert (ta - tb).abs().max().item() <= 1e-4 * scale, "%s %d" % (name, k)


def _run_steps(net, inp, tune, two_streams, steps=2):
    from paper_2503_23186_amd import StepRunner, cnnk
    for k, v in tune.items():
        cnnk.cnnk_tune(k, v)
    try:
        r = StepRunner(net.layers, net.slots, [p["shape"] for p in net.params], net.dtype, two_streams=two_streams)
        r.load(inp["x"], inp["labels"], inp["params"], inp["mom"])
        for _ in range(steps):
            r.step(0.1, 0.9, 1e-4)
        torch.cuda.synchronize()
    finally:
        for k in tune:
            cnnk.cnnk_tune(k, 0)
    return r


def _assert_same_bits(net, a, b):
    assert torch.equal(a.loss, b.loss)
    for s in range(1, len(net.slots)):
        assert torch.equal(a.act[s], b.act[s]), "activation %d" % s
        assert torch.equal(a.dact[s], b.dact[s]), "activation gradient %d" % s
    for k in range(len(net.params)):
        for name in ("grad", "param", "mom"):
            assert torch.equal(getattr(a, name)[k], getattr(b, name)[k]), "%s %d" % (name, k)


@pytest.mark.parametrize("name", ["mini_resnet", "mini_preact"])
def test_bn_backward_mask_from_y_equals_mask_recomputed_from_x(name):
    """Without a residual branch the step recomputes the ReLU mask from x instead of reading y
    (the forward kernel's own arithmetic on the same operands); handing y to every batch-norm
    backward call instead (tune key 9) must give the same bits everywhere, and the oracle's result."""
    net = getattr(WL, name)(batch=16, dtype="bf16", widths=(64, 128))
    inp = WL.make_inputs(net, 0, perturb_bn=True)
    a = _run_steps(net, inp, {}, two_streams=False)
    b = _run_steps(net, inp, {9: -1}, two_streams=False)
    _assert_same_bits(net, a, b)
    from paper_2503_23186_amd import cnnk
    cnnk.cnnk_tune(9, -1)
    try:
        inp2, runner, outs = run_both(net, 0, perturb_bn=True)
        check_step(net, inp2, runner, outs, TOL["bf16"])
    finally:
        cnnk.cnnk_tune(9, 0)


def test_weight_transposes_on_either_stream_give_the_same_bits():
    """With a second stream the weight transpositions of the data-gradient kernels run there beside
    the classifier head; tune key 12 keeps them on the main stream.  Same bits either way."""
    net = _two_stream_net()
    inp = WL.make_inputs(net, 0)
    a = _run_steps(net, inp, {}, two_streams=True, steps=3)
    b = _run_steps(net, inp, {12: -1}, two_streams=True, steps=3)
    _assert_same_bits(net, a, b)


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("C,size,batch", [(8, 1, 1), (24, 5, 3), (64, 7, 9), (136, 4, 2), (1024, 3, 2), (2048, 2, 1)])
def test_kept_relu_masks_give_the_gradients_that_y_gives(dtype, C, size, batch):
    """A batch norm with a residual input keeps its ReLU mask in the step; the entry point, which takes the mask from
    y, gives the same bits from the tensors that the step left: residual gradients written and accumulated."""
    from paper_2503_23186_amd import StepRunner, cnnk
    net = WL.Net("masks", batch, dtype)
    a = net.bn(net.conv(net.slot(batch, size, size, 3), C, 3, 1))
    r = net.bn(net.conv(a, C, 1, 1), relu=False)
    t = net.bn(net.conv(a, C, 1, 1), relu=True, res=r)
    for _ in range(2):
        t = net.bn(net.conv(t, C, 1, 1), relu=True, res=a)
    net.fc_loss(net.pool(t, "gap"))
    inp = WL.make_inputs(net, 23, perturb_bn=True)
    run = StepRunner(net.layers, net.slots, [p["shape"] for p in net.params], net.dtype)
    run.load(inp["x"], inp["labels"], inp["params"], inp["mom"])
    gains = [run.param[k].clone() for k in range(len(net.params))]
    run.step(0.1, 0.9, 0.0)
    checked = 0
    for i, L in enumerate(net.layers):
        if L["op"] != "bn" or L["res"] < 0:
            continue
        d = cnnk.bn_desc(batch, size, size, C, cnnk.BF16 if dtype == "bf16" else cnnk.F32, 1, 1e-5, 0.1)
        dx, dres = torch.empty_like(run.dact[L["x"]]), torch.empty_like(run.dact[L["res"]])
        dg, db = torch.empty(C, device="cuda:0"), torch.empty(C, device="cuda:0")
        need = int(cnnk.cnnk_bn_workspace_bytes(d))
        ws = torch.empty(need, dtype=torch.uint8, device="cuda:0")
        cnnk.cnnk_bn_relu_bwd(d, run.dact[L["y"]], run.act[L["x"]], run.act[L["y"]], gains[L["gamma"]], gains[L["beta"]],
                              run.bn_save[i][0], run.bn_save[i][1], dx, dres, 0, dg, db, ws, need,
                              torch.cuda.current_stream().cuda_stream)
        torch.cuda.synchronize()
        assert torch.equal(dx, run.dact[L["x"]]), (i, "dx")
        assert torch.equal(dg, run.grad[L["gamma"]].view(-1)) and torch.equal(db, run.grad[L["beta"]].view(-1)), i
        if L["res"] == r:
            assert torch.equal(dres, run.dact[r])
        checked += 1
    assert checked == 3


@pytest.mark.parametrize("two_streams", [True, False])
@pytest.mark.parametrize("widths,size,batch", [((64, 128), 8, 1), ((64, 128), 8, 21), ((64, 192), 16, 16), ((128, 512), 8, 37), ((72, 136), 8, 5)])
def test_batch_norms_that_add_up_the_partial_sums_agree_with_the_finalising_launch(widths, size, batch, two_streams):
    """A convolution's few partial sums per channel go straight to the batch norm behind it (widths of 64 channels; key 19 = -1
    keeps the launch that adds them up).  Both add in double and round once: statistics to a few ulp where the inputs are the
    same bits, the whole step to what a flipped bf16 rounding does."""
    net = WL.mini_resnet(batch=batch, dtype="bf16", size=size, widths=widths)
    inp = WL.make_inputs(net, 31)
    a = _run_steps(net, inp, {}, two_streams, steps=1)
    b = _run_steps(net, inp, {19: -1}, two_streams, steps=1)
    first = next(i for i, L in enumerate(net.layers) if L["op"] == "bn")
    assert torch.allclose(a.bn_save[first], b.bn_save[first], rtol=1e-6, atol=1e-7)
    for i, L in enumerate(net.layers):
        if L["op"] == "bn":
            assert (a.bn_save[i] - b.bn_save[i]).norm() <= 1e-2 * b.bn_save[i].norm(), i
            assert torch.isfinite(a.bn_save[i]).all()
    assert abs(a.loss.item() - b.loss.item()) <= 1e-2 * abs(b.loss.item())


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("widths,size,batch", [((8, 16), 8, 1), ((24, 40), 12, 5), ((64, 160), 16, 9)])
def test_sums_that_make_their_batch_norms_partial_sums_give_the_same_bits(widths, size, batch, dtype):
    """A sum in front of a batch norm leaves that one's partial sums, and its gradient goes to both summands in one launch; key 20 = -1
    keeps the launches apart.  The same rows, values and orders of summation: the same bits after two steps."""
    net = WL.mini_preact(batch=batch, dtype=dtype, size=size, widths=widths)
    inp = WL.make_inputs(net, 37, perturb_bn=True)
    a, b = _run_steps(net, inp, {}, True), _run_steps(net, inp, {20: -1}, True)
    _assert_same_bits(net, a, b)
    for i, L in enumerate(net.layers):
        if L["op"] == "bn":
            assert torch.equal(a.bn_save[i], b.bn_save[i]) and torch.equal(a.bn_running[i], b.bn_running[i])


def test_sums_of_many_channels_in_front_of_batch_norms():
    """The first of these sums is past the line beyond which it and the batch norm's partial sums are launches of their own, the second
    is not: the bits of both apart."""
    net = WL.mini_preact(batch=33, dtype="bf16", size=32, widths=(512, 1024))
    inp = WL.make_inputs(net, 37, perturb_bn=True)
    a, b = _run_steps(net, inp, {}, True), _run_steps(net, inp, {20: -1}, True)
    _assert_same_bits(net, a, b)


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("summand", ["a", "b"])
def test_sums_in_place(dtype, summand):
    """The sum of two convolutions' outputs, which nothing else reads, in the memory of one of them, its gradient likewise: the launches
    that take a sum apart from its batch norm and each gradient from the other, and the same bits as with memory of its own."""
    from paper_2503_23186_amd import StepRunner
    net = WL.mini_preact(batch=9, dtype=dtype, size=16, widths=(64, 160))
    inp = WL.make_inputs(net, 41, perturb_bn=True)
    runs = []
    for in_place in (False, True):
        r = StepRunner(net.layers, net.slots, [p["shape"] for p in net.params], net.dtype)
        sums = [L for L in net.layers if L["op"] == "add"]
        assert len(sums) == 2
        if in_place:
            for L in sums:
                r.buffers.act[L["y"]] = r.act[L[summand]].data_ptr()
                r.buffers.dact[L["y"]] = r.dact[L[summand]].data_ptr()
        r.load(inp["x"], inp["labels"], inp["params"], inp["mom"])
        for _ in range(2):
            r.step(0.1, 0.9, 1e-4)
        torch.cuda.synchronize()
        runs.append(r)
    a, b = runs
    assert torch.equal(a.loss, b.loss)
    for k in range(len(net.params)):
        assert torch.equal(a.grad[k], b.grad[k]) and torch.equal(a.param[k], b.param[k])
    for i, L in enumerate(net.layers):
        if L["op"] == "bn":
            assert torch.equal(a.bn_save[i], b.bn_save[i]) and torch.equal(a.bn_running[i], b.bn_running[i])


@pytest.mark.parametrize("group", [2, 5, 16])
def test_grouped_weight_gradients_give_the_same_bits(group):
    """Weight gradients forked onto the second stream one by one and several at a time, their reductions and updates
    in one launch: the same kernels and orders of summation, so the same bits after two steps."""
    from paper_2503_23186_amd import StepRunner, cnnk
    net = WL.mini_resnet(batch=224, dtype="bf16", size=32, widths=(32, 72))
    inp = WL.make_inputs(net, 29)
    out = []
    for g in (1, group):
        cnnk.cnnk_tune(17, g)
        try:
            run = StepRunner(net.layers, net.slots, [p["shape"] for p in net.params], net.dtype)
            run.load(inp["x"], inp["labels"], inp["params"], inp["mom"])
            for _ in range(2):
                run.step(0.1, 0.9, 1e-3)
            torch.cuda.synchronize()
        finally:
            cnnk.cnnk_tune(17, 0)
        out.append([t.clone() for t in run.param + run.mom + run.grad + [t for t in run.dact if t is not None]])
    assert uses_second_stream(net)
    for k, (a, b) in enumerate(zip(*out)):
        assert torch.equal(a, b), k


@pytest.mark.parametrize("group", [1, 2])
@pytest.mark.parametrize("dtype,k,stride,channels", [("bf16", 1, 1, 256), ("bf16", 3, 2, 256), ("bf16", 3, 1, 128), ("f32", 1, 1, 256)])
def test_layers_with_the_same_weights_take_those_that_the_step_began_with(dtype, k, stride, channels, group):
    """The second stream updates a layer's weights during the backward pass; the data gradient of a later layer with the
    same weights is the one-stream step's, bit for bit (a learning rate that moves every weight by its own size)."""
    from paper_2503_23186_amd import StepRunner, cnnk
    net = WL.Net("shared", 48, dtype)
    t = net.conv(net.slot(48, 32, 32, 3), channels, 3, 1)
    first = None
    for _ in range(3):
        t = net.bn(net.conv(t, channels, k, stride))
        conv = net.layers[-2]
        first = first or conv
        conv["w"] = first["w"]
    net.fc_loss(net.pool(t, "gap"))
    inp = WL.make_inputs(net, 31)
    assert uses_second_stream(net)
    out = []
    cnnk.cnnk_tune(17, group)
    try:
        for two in (False, True):
            run = StepRunner(net.layers, net.slots, [p["shape"] for p in net.params], net.dtype, two_streams=two)
            run.load(inp["x"], inp["labels"], inp["params"], inp["mom"])
            run.step(1e3, 0.9, 0.0)
            torch.cuda.synchronize()
            out.append(run)
    finally:
        cnnk.cnnk_tune(17, 0)
    for s in range(1, len(net.slots)):
        assert torch.equal(out[0].dact[s], out[1].dact[s]), "activation gradient %d" % s


def _steps_of(run, n):
    for _ in range(n):
        run.step(0.1, 0.9, 1e-4)


def _clones(run):
    return [t.clone() for t in run.param + run.mom + run.grad + [run.loss]]


def test_two_runners_on_two_streams_of_two_threads():
    """Steps of different streams share no stream: two host threads, each with its runner and its stream, leave the bits
    that either leaves alone; on one stream both use the same second one."""
    import threading
    from paper_2503_23186_amd import StepRunner
    net = _two_stream_net()
    inputs = [WL.make_inputs(net, s) for s in (37, 38)]
    make = lambda i: StepRunner(net.layers, net.slots, [p["shape"] for p in net.params], net.dtype)
    want = []
    for i in range(2):
        run = make(i)
        run.load(inputs[i]["x"], inputs[i]["labels"], inputs[i]["params"], inputs[i]["mom"])
        _steps_of(run, 6)
        torch.cuda.synchronize()
        want.append(_clones(run))
    runs, streams = [make(0), make(1)], [torch.cuda.Stream(), torch.cuda.Stream()]
    assert runs[0].aux_stream.cuda_stream == runs[1].aux_stream.cuda_stream and isinstance(runs[0].aux_stream, torch.cuda.Stream)
    for r, i in zip(runs, inputs):
        r.load(i["x"], i["labels"], i["params"], i["mom"])
    torch.cuda.synchronize()

    def work(k):
        with torch.cuda.stream(streams[k]):
            _steps_of(runs[k], 6)

    threads = [threading.Thread(target=work, args=(k,)) for k in range(2)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    torch.cuda.synchronize()
    assert len({runs[0].aux_stream.cuda_stream, runs[1].aux_stream.cuda_stream} | {s.cuda_stream for s in streams}) == 4
    for r, w in zip(runs, want):
        for k, (a, b) in enumerate(zip(_clones(r), w)):
            assert torch.equal(a, b), k


def test_captured_step_beside_steps_of_another_stream():
    """A step captured into a graph on a stream of its own, while another runner's steps are enqueued on another stream:
    they run at once and are no part of the graph.  Every replay, with eager work in between, is the eager step."""
    from paper_2503_23186_amd import StepRunner
    net = _two_stream_net()
    inputs = [WL.make_inputs(net, s) for s in (41, 42)]
    eager, taken, other, alone = (StepRunner(net.layers, net.slots, [p["shape"] for p in net.params], net.dtype) for _ in range(4))
    for r, i in ((eager, 0), (taken, 0), (other, 1), (alone, 1)):
        r.load(inputs[i]["x"], inputs[i]["labels"], inputs[i]["params"], inputs[i]["mom"])
    _steps_of(alone, 3)
    side, graph = torch.cuda.Stream(), torch.cuda.CUDAGraph()
    torch.cuda.synchronize()
    with torch.cuda.graph(graph, capture_error_mode="thread_local"):
        _steps_of(taken, 1)
        with torch.cuda.stream(side):
            _steps_of(other, 3)
    side.synchronize()
    for k, (a, b) in enumerate(zip(_clones(other), _clones(alone))):
        assert torch.equal(a, b), k
    for replay in range(3):
        graph.replay()
        _steps_of(eager, 1)
        torch.cuda.synchronize()
        for k, (a, b) in enumerate(zip(_clones(taken), _clones(eager))):
            assert torch.equal(a, b), (replay, k)
    for k, (a, b) in enumerate(zip(_clones(other), _clones(alone))):
        assert torch.equal(a, b), k
