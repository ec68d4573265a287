"""GPU tests of the row-tile path at the edges of what it takes: one hidden layer, the widest
layers it accepts (one critic at a time), heads of 1 and 32 actions, batches below, at and
past its tiles, and the batch at which networks with the row split change paths."""
import numpy as np
import pytest
import torch   # before the library: the first of the two to load chooses the HIP runtime

import synth
from synth.workloads import Workload

from .helpers import log, make_gpu
from .test_gpu_parity import BF16_LOSS_TOL, FP32_TOL, FUSED_BF16, RAGGED, RAGGED_TD3, teacher_forced

pytestmark = pytest.mark.gpu

WIDE = Workload("wide_rows", "sac", 376, 32, (512, 480), 200, 4000, "fp32", 10, target_entropy=-32.0)
CASES = [
    RAGGED.replace(name="one_layer", hidden=(32,), act_dim=1, batch=1),
    RAGGED.replace(name="one_wide_layer_td3", algo="td3", hidden=(416,), batch=33, learn_alpha=False, alpha_init=0.0),
    WIDE,                                                        # one critic at a time
    WIDE.replace(name="wide_rows_bf16", prec="bf16", hidden=(480, 512, 96)),
    RAGGED_TD3.replace(name="deep_td3", hidden=(40, 300, 64, 33), obs_dim=65, act_dim=33, batch=97),
    FUSED_BF16.replace(name="tiles64", batch=16385, hidden=(128, 128)),   # 64-row tiles, a ragged last one
]


@pytest.mark.parametrize("w", CASES, ids=[w.name for w in CASES])
def test_row_path_teacher_forced(w):
    """Every gradient tensor, Adam's moments and the losses of one step from the oracle's state
    (bounds as for the other teacher-forced tests: 1e-4 in float32, 1e-3 in bfloat16)."""
    log("row path %s" % w.name)
    g = make_gpu(w)
    g.buffer_push(*synth.workload_rows(w, 0, 1000, 0))
    g.profile_enable(True, 100)
    g.update(1)
    names = {s["name"] for s in g.profile_read()}
    g.close()
    assert names == {"row_step", "row_wgrad", "row_adam"}, names
    bf16 = w.prec == "bf16"
    teacher_forced(w, 4000, steps_before=1, n_steps=2, tol_grad=1e-3 if bf16 else FP32_TOL,
                   tol_loss=BF16_LOSS_TOL if bf16 else FP32_TOL)


# Batches at which the joint launch of actor and critics needs a larger workspace of
# weight-gradient slices than the launches of either added up.
JOINT = [
    Workload("sac_fp32_32k", "sac", 17, 6, (256, 256), 32768, 40000, "fp32", 0, target_entropy=-6.0),
    Workload("sac_bf16_64k", "sac", 17, 6, (256, 256), 65536, 70000, "bf16", 0, target_entropy=-6.0),
    Workload("td3_fp32_16k", "td3", 111, 8, (400, 300), 16384, 40000, "fp32", 0, learn_alpha=False, alpha_init=0.0),
]


@pytest.mark.parametrize("w", JOINT, ids=[w.name for w in JOINT])
def test_joint_weight_gradients_teacher_forced(w):
    """Steps that take the actor's and the critics' weight gradients in one launch, against
    the oracle (bounds as for the other teacher-forced tests)."""
    log("joint weight gradients %s" % w.name)
    bf16 = w.prec == "bf16"
    teacher_forced(w, 4000, steps_before=1, n_steps=1, tol_grad=1e-3 if bf16 else FP32_TOL,
                   tol_loss=BF16_LOSS_TOL if bf16 else FP32_TOL)


@pytest.mark.parametrize("b", [500, 1024, 1500])
def test_set_batch_across_the_path_change_bit_exact(b):
    """A context created for 2048 rows, having run steps there, computes at batch b what a
    context created with b does from the same state, whichever path either batch takes."""
    w = FUSED_BF16
    out = []
    state = None
    for created in (2048, b):
        g = make_gpu(w.replace(batch=created))
        g.buffer_push(*synth.workload_rows(w, 0, 5000, 0))
        keys = ["actor", "critic1", "critic2", "tcritic1", "tcritic2", "log_alpha"]
        keys += [m + k for m in ("m_", "v_") for k in ("actor", "critic1", "critic2", "log_alpha")]
        if state is None:
            g.update(2)
            state = {k: g.read_params(k) for k in keys}
            g.set_batch(b)
        else:
            for k in keys:
                g.write_params(k, state[k])
            g.set_step(2)
        g.update(2)
        obs = synth.workload_rows(w, 0, 40, 3)[0]
        out.append({k: g.read_params(k) for k in keys})
        out[-1].update(rec=g.read_losses(3, 2), idx=g.debug_indices(), act=g.act(obs, True, 5),
                       da=g.debug_rows("daction"), batch=np.concatenate([np.ravel(x) for x in g.debug_batch()]))
        g.close()
    for k in out[0]:
        assert np.array_equal(out[0][k], out[1][k]), k


@pytest.mark.parametrize("prec", ["fp32", "bf16"])
@pytest.mark.parametrize("obs_dim", [5, 8, 31, 260])
def test_layered_actions_from_any_alignment(prec, obs_dim):
    """The layer-by-layer action call (a layer past the row tiles) reads rows of four-column
    multiples on 16 bytes whole and others by the element: the same actions."""
    from paper_2312_06126_amd import Spz
    g = Spz(obs_dim, 3, (544,), 256, dict(algo="sac", gemm_prec=prec, capacity=256), 1)
    obs = np.random.default_rng(0).standard_normal((77, obs_dim)).astype(np.float32)
    out = []
    for shift in (0, 1):
        buf = torch.zeros(obs.size + 4, device="cuda")
        buf[shift:shift + obs.size] = torch.from_numpy(obs.ravel()).cuda()
        act = torch.empty(77, 3, device="cuda")
        torch.cuda.synchronize()
        g.act_noalloc(buf.data_ptr() + 4 * shift, 77, act.data_ptr())
        torch.cuda.synchronize()
        out.append(act.cpu().numpy())
    host = g.act(obs)
    g.close()
    assert np.array_equal(out[0], out[1]) and np.array_equal(out[0], host)


@pytest.mark.parametrize("negative", [False, True], ids=["pos", "neg"])
@pytest.mark.parametrize("prec,hidden,batch", [
    ("bf16", (64,), 300), ("bf16", (200, 120), 300), ("bf16", (256, 256), 2000), ("fp32", (200, 120), 300),
    ("bf16", (256, 256), 300), ("bf16", (544, 100), 300), ("bf16", (1024,), 300), ("bf16", (512, 640), 3000)])
def test_nan_reaches_actions_and_loss_record(prec, hidden, batch, negative):
    """A NaN of either sign, in an observation column or in a critic's first bias, makes the
    actions that depend on it NaN and sets the step's non-finite flag."""
    nan = np.uint32(0xFFC00000 if negative else 0x7FC00000).reshape(1).view(np.float32)[0]
    w = RAGGED.replace(name="nan", hidden=hidden, batch=batch, prec=prec)
    rows = [np.array(x) for x in synth.workload_rows(w, 0, 2000, 0)]
    g = make_gpu(w)
    g.buffer_push(*rows)
    p = g.read_params("critic1")
    p[(w.obs_dim + w.act_dim) * hidden[0] + 5] = nan
    g.write_params("critic1", p)
    g.update(1)
    assert g.read_losses(1, 1)[0, 6] == 1.0
    g.close()
    rows[0][:, 3] = nan
    g = make_gpu(w)
    g.buffer_push(*rows)
    assert np.isnan(g.act(rows[0][:33])).all()
    g.update(1)
    assert g.read_losses(1, 1)[0, 6] == 1.0
    g.close()


@pytest.mark.parametrize("algo", ["sac", "td3"])
@pytest.mark.parametrize("prec,hidden,n_streams,ordering", [
    ("fp32", (64, 64), 1, "snapshot"), ("fp32", (64, 64), 2, "sequential"), ("bf16", (200, 120), 1, "snapshot"),
    ("bf16", (256, 256), 1, "snapshot"), ("fp32", (544,), 1, "sequential")])
def test_debug_reads_before_the_first_step_are_zero(algo, prec, hidden, n_streams, ordering):
    base = RAGGED if algo == "sac" else RAGGED_TD3
    g = make_gpu(base.replace(name="fresh", prec=prec, hidden=hidden, batch=300, ordering=ordering), n_streams=n_streams)
    arrays = list(g.debug_batch()) + [g.debug_rows(k) for k in ("daction", "td_target", "q", "qpi")]
    assert not any(np.any(a) for a in arrays) and not g.debug_indices().any()
    g.close()


@pytest.mark.parametrize("hidden", [(64, 40), (544, 40)], ids=["row_tiles", "layers"])
@pytest.mark.parametrize("prec", ["fp32", "bf16"])
def test_adam_and_polyak_round_as_written(prec, hidden):
    """Moments and targets of a step, bit for bit: one rounding of (1 - beta1) g + fl(beta1 m),
    of fl((1 - beta2) g) g + fl(beta2 v) and of tau p + fl((1 - tau) target), on both paths.
    The products are exact in the 64-bit significands used here; a sum that rounds twice there
    would need its last 40 bits to hit the tie of the first rounding."""
    w = RAGGED.replace(name="adam", hidden=hidden, batch=300, prec=prec)
    g = make_gpu(w)
    g.buffer_push(*synth.workload_rows(w, 0, 2000, 0))
    g.update(3)
    keys = [m + k for m in ("", "m_", "v_", "t") for k in ("actor", "critic1", "critic2") if m + k != "tactor"]
    old = {k: g.read_params(k) for k in keys}
    g.update(1)
    hp = w.hparams()
    one, f32, wide = np.float32(1), np.float32, np.longdouble
    assert np.finfo(wide).nmant >= 63
    b1, b2, tau = (f32(hp.get(k, d)) for k, d in (("beta1", 0.9), ("beta2", 0.999), ("tau", 0.005)))
    for k in ("actor", "critic1", "critic2"):
        grad = g.read_params("g_" + k)
        m = (wide(one - b1) * grad.astype(wide) + (b1 * old["m_" + k]).astype(wide)).astype(f32)
        v = (((one - b2) * grad).astype(wide) * grad.astype(wide) + (b2 * old["v_" + k]).astype(wide)).astype(f32)
        assert np.array_equal(g.read_params("m_" + k), m), k
        assert np.array_equal(g.read_params("v_" + k), v), k
        if k != "actor":
            t = (wide(tau) * g.read_params(k).astype(wide) + ((one - tau) * old["t" + k]).astype(wide)).astype(f32)
            assert np.array_equal(g.read_params("t" + k), t), k
    g.close()


# Networks and batches on either side of the lines between the paths, where the chip is left
# idle by too few tiles (float32) or 512-wide weights pass through too many CUs (bfloat16).
F400 = Workload("fp32_400_300_seq", "sac", 376, 6, (400, 300), 3100, 20000, "fp32", 10, target_entropy=-6.0,
                ordering="sequential")
B512 = Workload("bf16_512_x3", "sac", 376, 17, (512, 512, 512), 17000, 20000, "bf16", 10, target_entropy=-17.0)
SIDES = [(F400, 300, False), (F400, 3071, False), (F400, 3072, True), (F400.replace(ordering="snapshot"), 300, True),
         (F400.replace(algo="td3", learn_alpha=False, alpha_init=0.0, ordering="snapshot"), 300, False),
         (B512, 1023, False), (B512, 1024, True), (B512, 16384, True), (B512, 16385, False)]


@pytest.mark.parametrize("w,b,rows", SIDES, ids=["%s-%s-%s-%d" % (w.name, w.algo, w.ordering, b) for w, b, _ in SIDES])
def test_path_of_a_batch_and_its_results(w, b, rows):
    """The path a batch takes, and the same results from a context created for more rows (which
    has run another batch, on the other path where there is one) as from one created for b."""
    out = []
    for created in (w.batch, b):
        g = make_gpu(w.replace(batch=created))
        g.buffer_push(*synth.workload_rows(w, 0, 5000, 0))
        if created != b:
            keep = {k: g.read_params(k) for k in ("actor", "critic1", "critic2", "tcritic1", "tcritic2")}
            g.update(1)
            g.set_batch(2000)
            g.update(1)
            for k in keep:
                g.write_params(k, keep[k])
            for k in ("actor", "critic1", "critic2", "log_alpha"):
                for m in ("m_", "v_"):
                    g.write_params(m + k, np.zeros(g.param_count(m + k), np.float32))
            g.write_params("log_alpha", np.full(1, np.log(w.alpha_init) if w.algo == "sac" else 0.0, np.float32))
            if w.algo == "td3":
                g.write_params("tactor", keep["actor"])
            g.set_batch(b)
            g.set_step(0)
        g.profile_enable(True, 1000)
        g.update(2)
        assert ("row_step" in {s["name"] for s in g.profile_read()}) == rows
        out.append({k: g.read_params(k) for k in ("actor", "critic1", "critic2", "tcritic1", "m_critic2", "log_alpha")})
        out[-1].update(rec=g.read_losses(1, 2), act=g.act(synth.workload_rows(w, 0, 70, 3)[0]), da=g.debug_rows("daction"))
        g.close()
    for k in out[0]:
        assert np.array_equal(out[0][k], out[1][k]), k


@pytest.mark.parametrize("n_streams", [1, 2])
def test_debug_reads_after_a_larger_batch_was_set(n_streams):
    """A context whose layer buffers hold fewer rows than the batch now set: debug reads give the
    last step's rows and end with the buffers."""
    g = make_gpu(F400, n_streams=n_streams)
    g.buffer_push(*synth.workload_rows(F400, 0, 5000, 0))
    g.set_batch(200)
    g.update(1)
    small = [np.array(x) for x in g.debug_batch()] + [g.debug_rows("daction")]
    g.set_batch(3100)
    large = list(g.debug_batch()) + [g.debug_rows("daction")]
    g.close()
    for a, b in zip(small, large):
        assert len(b) == 3100 and np.array_equal(a, b[:200])


@pytest.mark.parametrize("obs_dim,hidden,created", [(17, (400, 300), 1000), (17, (400, 300), 20000), (376, (256, 256), 700),
                                                    (376, (400, 300), 6000), (13, (64, 64), 300)])
def test_float32_actions_on_either_path(obs_dim, hidden, created):
    """float32 action calls from one observation to two rounds of tiles, on both sides of each
    line between the paths: spz_act (in chunks) and spz_act_noalloc give the same bits, both
    within float32 rounding of the actor in 64 bits (the bound of the sampler parity test)."""
    from oracle import Oracle
    w = RAGGED.replace(name="act", obs_dim=obs_dim, hidden=hidden, batch=created)
    g = make_gpu(w)
    o = Oracle(w.obs_dim, w.act_dim, w.hidden, w.batch, w.hparams(), 1)
    obs = np.random.default_rng(5).standard_normal((13000, obs_dim)).astype(np.float32)
    ref = o.act(obs.astype(np.float64), True, 9)
    dev = torch.from_numpy(obs).cuda()
    for n in (1, 33, 2047, 2048, 4095, 4096, 8192, 8225, 13000):
        out = torch.empty(n, w.act_dim, device="cuda")
        torch.cuda.synchronize()
        g.act_noalloc(dev.data_ptr(), n, out.data_ptr(), True, 9)
        torch.cuda.synchronize()
        host = g.act(obs[:n], True, 9)
        assert np.array_equal(host, out.cpu().numpy()), n
        assert np.abs(host - ref[:n]).max() <= 1e-5, n
    g.close()


@pytest.mark.parametrize("hidden", [(32, 32), (64, 64), (100, 70), (128, 128), (300, 200)])
def test_read_params_gives_what_was_written(hidden):
    """On both sides of the sizes that are copied directly, for every network and its moments."""
    g = make_gpu(RAGGED_TD3.replace(name="io", hidden=hidden, batch=64))
    rng = np.random.default_rng(2)
    keys = ["actor", "critic1", "critic2", "tactor", "tcritic1", "tcritic2", "m_actor", "v_critic2"]
    want = {k: rng.standard_normal(g.param_count(k)).astype(np.float32) for k in keys}
    for k in keys:
        g.write_params(k, want[k])
    for k in keys:
        assert np.array_equal(g.read_params(k), want[k]), k
    g.close()


@pytest.mark.parametrize("prec,hidden", [("fp32", (64, 64)), ("fp32", (400, 300)), ("bf16", (400, 300))])
def test_first_action_call_in_a_captured_graph(prec, hidden):
    """A new context's first launch is an action call that is being captured; its replays, with the
    context's own eager calls between them, give the eager call's actions."""
    w = RAGGED.replace(name="capture", prec=prec, hidden=hidden, batch=300)
    obs = torch.randn(90, w.obs_dim, device="cuda")
    act = torch.zeros(90, w.act_dim, device="cuda")
    torch.cuda.synchronize()
    g = make_gpu(w)
    graph, stream = torch.cuda.CUDAGraph(), torch.cuda.Stream()
    with torch.cuda.graph(graph, stream=stream):
        g.act_noalloc(obs.data_ptr(), 90, act.data_ptr(), True, 4, torch.cuda.current_stream())
    for _ in range(3):
        act.zero_()
        graph.replay()
        torch.cuda.synchronize()
        assert np.array_equal(act.cpu().numpy(), g.act(obs.cpu().numpy(), True, 4))
    g.close()


@pytest.mark.parametrize("algo,obs_dim,act_dim,hidden,batch", [
    ("sac", 376, 6, (400, 300), 257), ("sac", 300, 31, (480, 64, 512), 1000), ("sac", 376, 1, (416,), 33),
    ("sac", 45, 3, (500, 330, 33), 1), ("sac", 7, 2, (480, 480, 480), 640)])
def test_both_paths_agree(algo, obs_dim, act_dim, hidden, batch):
    """float32 networks with a weight of more than 150000 elements (so the wide layers of the
    fourth stand next to each other), whose small batches take row tiles on one stream and go
    layer by layer from graphs on two: one step from the same state. Hidden layers and policy
    heads sum in the same order on both paths: log-probabilities have the same bits. The critics'
    one-column output and the gradients differ by the order of float32 sums over up to 1000
    terms, about sqrt(1000) 2^-24 = 1.9e-6 of a tensor's norm at most (measured: 2.5e-7). Two
    optimizer steps later an element whose gradient is of that size may have moved the other way
    (measured: 7e-8 of the loss record's norm)."""
    from paper_2312_06126_amd import Spz
    w = RAGGED.replace(name="both", algo=algo, obs_dim=obs_dim, act_dim=act_dim, hidden=hidden, batch=batch)
    out = []
    for n_streams, graphs in ((1, False), (2, True)):
        g = Spz(obs_dim, act_dim, hidden, batch, dict(w.hparams(), graphs=graphs), 1, n_streams=n_streams)
        g.buffer_push(*synth.workload_rows(w, 0, 3000, 0))
        if n_streams == 1:
            g.profile_enable(True, 100)
        g.update(1)
        if n_streams == 1:
            assert {s["name"] for s in g.profile_read()} == {"row_step", "row_wgrad", "row_adam"}
        out.append({k: g.read_params("g_" + k).astype(np.float64) for k in ("actor", "critic1", "critic2", "log_alpha")})
        out[-1].update(rec=g.read_losses(1, 1), q=g.debug_rows("q"), qpi=g.debug_rows("qpi"), logpi=g.debug_rows("logpi"))
        g.update(2)
        out[-1]["later"] = g.read_losses(2, 2)
        g.profile_enable(True, 100)   # (eager while timing)
        g.update(1)
        assert ("row_step" in {s["name"] for s in g.profile_read()}) == (n_streams == 1)
        g.close()
    a, b = out
    assert np.array_equal(a["logpi"], b["logpi"])
    for k, tol in dict(q=2e-6, qpi=2e-6, rec=2e-6, actor=2e-6, critic1=2e-6, critic2=2e-6, log_alpha=2e-6,
                       later=1e-5).items():
        assert np.linalg.norm(a[k] - b[k]) <= tol * np.linalg.norm(b[k]), k
