"""The one-launch kernels that take any layer widths -- the resident trainer kernel (bf16) and the fp32 kernels --
against the per-layer kernels of the same instance (gmi_set_fusion 0), at the sizes where their tiling can go wrong:
rows around the tile heights, widths around the 32- and 64-wide blocks, one to four hidden layers."""
import numpy as np
import pytest
import torch

from workloads import synthetic as syn
from gpu_util import rel_l2, rel_max

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def g():
    import paper_2206_08482_amd as m
    return m


@pytest.fixture(scope="module")
def inst(g):
    h = g.gmi_create()
    yield h
    g.gmi_destroy(h)


def _setup(g, inst, obs, act, hidden, dtype, T, N, rows, seed=3):
    from paper_2206_08482_amd.runner import RolloutBuffers
    dev = torch.device("cuda:0")
    theta = torch.tensor(syn.make_model_params(obs, act, hidden, seed, policy_head_scale=0.5), device=dev)
    desc = g.model_desc(obs, act, list(hidden), g.dtype_code(dtype), rows)
    nb = g.gmi_model_shadow_bytes(desc)
    shadow = torch.zeros(nb, dtype=torch.uint8, device=dev) if nb else None
    m, v = torch.zeros_like(theta), torch.zeros_like(theta)
    rb = RolloutBuffers(T, N, obs, act, dev)
    b = syn.make_rollout_batch(T, N, obs, act, seed=seed)
    for k in ("obs", "act", "logp", "val", "rew", "done"):
        getattr(rb, k).copy_(torch.tensor(b[k]))
    rb.adv.copy_(torch.tensor(b["val"])); rb.ret.copy_(torch.tensor(b["rew"]))
    torch.cuda.synchronize()
    model = g.gmi_model_bind(inst, desc, theta, shadow, m, v)
    g.gmi_model_refresh_shadow(inst, model)
    buf = g.gmi_buffer_bind(inst, rb.desc(0, N))
    return model, buf, (theta, shadow, m, v, rb)


def _gradients(g, inst, model, buf, n_par, T, N, rows, fused):
    g.gmi_set_fusion(inst, fused)
    idx = torch.tensor(np.random.default_rng(1).permutation(T * N)[:rows].astype(np.int32), device="cuda:0")
    hp = g.ppo_hparams(clip=0.2, c_v=0.5, c_e=0.01, minibatch=rows)
    grad, stats = torch.zeros(n_par, device="cuda:0"), torch.zeros(5, device="cuda:0")
    torch.cuda.synchronize()
    g.ppo_gradient(inst, model, buf, hp, idx, rows, grad, stats)
    g.gmi_sync(inst)
    g.gmi_set_fusion(inst, 1)
    return grad.cpu().numpy(), stats.cpu().numpy()


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("obs,act,hidden", [
    (45, 12, (128, 128)), (60, 8, (256, 128, 64)), (3, 1, (32,)), (64, 32, (33, 65)), (5, 23, (100, 48, 32)),
    (130, 22, (256, 32)), (44, 18, (300, 200, 200)), (70, 11, (400, 128, 128, 64)), (251, 16, (100, 100)),
    (197, 14, (512, 200, 100)), (16, 4, (48,))])
@pytest.mark.parametrize("rows", [1, 31, 33, 130, 4097, 16500])
def test_gradient_equals_the_per_layer_kernels(g, inst, obs, act, hidden, dtype, rows):
    T, N = (1, rows) if rows < 100 else (2, (rows + 1) // 2)
    model, buf, keep = _setup(g, inst, obs, act, hidden, dtype, T, N, rows)
    n = keep[0].numel()
    a, sa = _gradients(g, inst, model, buf, n, T, N, rows, 1)
    b, sb = _gradients(g, inst, model, buf, n, T, N, rows, 0)
    assert np.isfinite(a).all()
    tol = 1e-5 if dtype == "f32" else 5e-3          # bf16: same roundings, other order of the fp32 sums
    if rows < 100 and dtype == "bf16":
        tol = 2e-2                                   # few rows: one activation that rounds the other way is not averaged
    assert rel_l2(a, b) <= tol, rel_l2(a, b)
    assert rel_max(a, b) <= 4 * tol, rel_max(a, b)
    assert np.allclose(sa, sb, rtol=tol, atol=tol)
    g.gmi_buffer_destroy(buf)
    g.gmi_model_destroy(model)


@pytest.mark.parametrize("obs,act,hidden,rows", [
    (60, 8, (256, 128, 64), 63501),              # activations kept in LDS, 252 MB of them stored
    (108, 21, (400, 200, 100), 37201),           # read back from memory, 252 MB
    (211, 20, (512, 512, 256, 128), 30001),      # 369 MB: the weight gradients alone stream
    (211, 20, (512, 512, 256, 128), 26753),      # 128 rows per workgroup, a second round five eighths full, a last tile of one row
    (211, 20, (512, 512, 512, 256), 32897),      # .., two full rounds and a third of two workgroups with one row
])
def test_gradient_of_large_minibatches(g, inst, obs, act, hidden, rows):
    """Beyond the memory-side cache activations and gradients are stored and read as streams.  The second of two minibatches, which finds the
    first one's lines wherever they were left, against the per-layer kernels; the band as above (same roundings, other order of sums)."""
    model, buf, keep = _setup(g, inst, obs, act, hidden, "bf16", 2, rows // 2 + 200, rows)
    n, total = keep[0].numel(), 2 * (rows // 2 + 200)
    hp = g.ppo_hparams(clip=0.2, c_v=0.5, c_e=0.01, minibatch=rows)
    idx = [torch.tensor(np.random.default_rng(s).permutation(total)[:rows].astype(np.int32), device="cuda:0") for s in (1, 2)]
    out = []
    for fused in (1, 0):
        grads, stats = [torch.zeros(n, device="cuda:0") for _ in idx], torch.zeros(5, device="cuda:0")
        torch.cuda.synchronize()
        g.gmi_set_fusion(inst, fused)
        for i, gr in zip(idx, grads):
            g.ppo_gradient(inst, model, buf, hp, i, rows, gr, stats)
        g.gmi_sync(inst)
        out.append(([v.cpu().numpy() for v in grads], stats.cpu().numpy()))
    g.gmi_set_fusion(inst, 1)
    (a, sa), (b, sb) = out
    assert all(np.isfinite(v).all() for v in a) and not np.array_equal(a[0], a[1])
    for x, y in zip(a, b):
        assert rel_l2(x, y) <= 5e-3 and rel_max(x, y) <= 2e-2, (rel_l2(x, y), rel_max(x, y))
    assert np.allclose(sa, sb, rtol=5e-3, atol=5e-3)
    g.gmi_buffer_destroy(buf)
    g.gmi_model_destroy(model)


@pytest.mark.parametrize("obs,act,hidden,reads_back", [(60, 8, (256, 128, 64), False), (108, 21, (400, 200, 100), True)])
def test_stated_bytes_count_activations_read_back_where_they_are(g, inst, obs, act, hidden, reads_back):
    rows = 512
    model, buf, keep = _setup(g, inst, obs, act, hidden, "bf16", 2, rows // 2, rows)
    cls = [g.gmi_profile_class_name(c) for c in range(g.gmi_profile_classes())].index("chain_train")
    g.gmi_profile_enable(inst, 1 << cls)
    _gradients(g, inst, model, buf, keep[0].numel(), 2, rows // 2, rows, 1)
    launches, stated = g.gmi_profile_read(inst, cls)[1], g.gmi_profile_work(inst, cls)[1]
    g.gmi_profile_enable(inst, 0)
    want = rows * (6 * obs + 4 * (act + 3))      # observations read, their bf16 copy written; scalars of a sample
    for out in (act, 1):
        dims = (obs, *hidden, out)
        for l, (i, o) in enumerate(zip(dims, dims[1:])):
            want += 2 * i * o * (2 if l else 1) + 2 * rows * o + (2 * rows * i * (2 if reads_back else 1) if l else 0)
    assert launches == 1 and stated == want
    g.gmi_buffer_destroy(buf)
    g.gmi_model_destroy(model)


@pytest.mark.parametrize("obs,hidden", [(211, (512, 512, 256, 128)), (108, (400, 200, 100))])
@pytest.mark.parametrize("act", [1, 2, 3, 4, 5, 7, 31, 32])
@pytest.mark.parametrize("rows", [1, 3, 301])
def test_gradient_of_every_remainder_of_the_actions(g, inst, obs, act, hidden, rows):
    """The row-tile trainer kernel reads a sample's actions four at a time (fewer than 4 actions in all: it does not run)."""
    model, buf, keep = _setup(g, inst, obs, act, hidden, "bf16", 1, rows, rows)
    n = keep[0].numel()
    a, sa = _gradients(g, inst, model, buf, n, 1, rows, rows, 1)
    b, sb = _gradients(g, inst, model, buf, n, 1, rows, rows, 0)
    tol = 5e-3 if rows > 100 else 2e-2              # as above
    assert rel_l2(a, b) <= tol, rel_l2(a, b)
    assert rel_max(a, b) <= 4 * tol, rel_max(a, b)
    assert np.allclose(sa, sb, rtol=tol, atol=tol)
    g.gmi_buffer_destroy(buf)
    g.gmi_model_destroy(model)


@pytest.mark.parametrize("obs,hidden", [(60, (256, 128, 64)), (23, (256, 128, 64)), (108, (400, 200, 100)), (108, (200, 400, 100)),
                                        (211, (512, 512, 256, 128)), (211, (512, 512, 512, 256))])
@pytest.mark.parametrize("act,N", [(1, 1), (1, 3), (2, 1), (3, 1), (3, 2)])
def test_gradient_does_not_depend_on_what_lies_between_the_slots(g, inst, obs, hidden, act, N):
    """Columns of a wider experience array: the row-tile trainer kernel reads actions four at a time, at the array's start beyond a
    sample's own.  What lies in the other columns -- NaN, infinities -- does not reach the gradient: bit for bit that with zeros."""
    from paper_2206_08482_amd.runner import RolloutBuffers
    T, ld = 4, N + 5
    dev = torch.device("cuda:0")
    theta = torch.tensor(syn.make_model_params(obs, act, hidden, 3, policy_head_scale=0.5), device=dev)
    desc = g.model_desc(obs, act, list(hidden), g.dtype_code("bf16"), T * N)
    shadow = torch.zeros(g.gmi_model_shadow_bytes(desc), dtype=torch.uint8, device=dev)
    b = syn.make_rollout_batch(T, N, obs, act, seed=3)
    b.update(adv=b["val"], ret=b["rew"])
    torch.cuda.synchronize()
    model = g.gmi_model_bind(inst, desc, theta, shadow, torch.zeros_like(theta), torch.zeros_like(theta))
    g.gmi_model_refresh_shadow(inst, model)
    out = []
    for other in (0.0, float("nan"), float("inf")):
        rb = RolloutBuffers(T, ld, obs, act, dev)
        for k in ("obs", "act", "logp", "val", "rew", "adv", "ret"):
            getattr(rb, k).fill_(other)
            getattr(rb, k)[:, :N].copy_(torch.tensor(b[k]))
        torch.cuda.synchronize()
        buf = g.gmi_buffer_bind(inst, rb.desc(0, N))
        out.append(_gradients(g, inst, model, buf, theta.numel(), T, N, T * N, 1))
        g.gmi_buffer_destroy(buf)
    g.gmi_model_destroy(model)
    for grad, stats in out:
        assert np.isfinite(grad).all() and np.array_equal(grad, out[0][0]) and np.array_equal(stats, out[0][1])


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("obs,act,hidden,rows", [(45, 12, (128, 128), 3001), (17, 6, (64, 64), 700), (8, 2, (32, 32), 130),
                                                 (44, 18, (300, 200, 200), 1500)])
def test_gradient_on_eight_compute_units_equals_the_per_layer_kernels(g, obs, act, hidden, rows, dtype):
    """Four workgroups per net, each with several tiles."""
    from paper_2206_08482_amd.instances import cu_masks
    masked = g.gmi_create(cu_masks(256, [8])[0])
    N = (rows + 1) // 2
    model, buf, keep = _setup(g, masked, obs, act, hidden, dtype, 2, N, rows)
    n = keep[0].numel()
    a, sa = _gradients(g, masked, model, buf, n, 2, N, rows, 1)
    b, sb = _gradients(g, masked, model, buf, n, 2, N, rows, 0)
    tol = 1e-5 if dtype == "f32" else 5e-3          # as on the whole device, above
    assert rel_l2(a, b) <= tol, rel_l2(a, b)
    assert rel_max(a, b) <= 4 * tol, rel_max(a, b)
    assert np.allclose(sa, sb, rtol=tol, atol=tol)
    g.gmi_buffer_destroy(buf)
    g.gmi_model_destroy(model)
    g.gmi_destroy(masked)


@pytest.mark.parametrize("cus,rows", [(8, 95), (8, 96), (8, 512), (8, 513), (80, 959), (80, 2000), (80, 2560)])
def test_gradient_at_the_line_between_the_trainer_kernels(g, cus, rows):
    """60:256:128:64:8 on few compute units: both sides of the rule between the resident and the row-tile kernel."""
    from paper_2206_08482_amd.instances import cu_masks
    masked = g.gmi_create(cu_masks(256, [cus])[0])
    N = (rows + 1) // 2
    model, buf, keep = _setup(g, masked, 60, 8, (256, 128, 64), "bf16", 2, N, rows)
    a, sa = _gradients(g, masked, model, buf, keep[0].numel(), 2, N, rows, 1)
    b, sb = _gradients(g, masked, model, buf, keep[0].numel(), 2, N, rows, 0)
    assert np.isfinite(a).all() and rel_l2(a, b) <= 5e-3 and rel_max(a, b) <= 2e-2      # the bf16 band above
    assert np.allclose(sa, sb, rtol=5e-3, atol=5e-3)
    g.gmi_buffer_destroy(buf)
    g.gmi_model_destroy(model)
    g.gmi_destroy(masked)


@pytest.mark.parametrize("obs,act,hidden,n,shift", [
    (1, 1, [32], 1, 0),                       # one column, one action, one row
    (45, 12, [128, 128], 31, 0),              # rows of an odd length: 16-byte pieces span two rows
    (45, 12, [128, 128], 65, 1),              # ... of an array that is not 16-byte aligned
    (60, 8, [256, 128, 64], 33, 1),
    (60, 8, [256, 128, 64], 8193, 0),         # more 32-row tiles than fit at once: 64-row tiles
    (45, 12, [128, 128], 32801, 1),           # enough rows for 128-row tiles
    (108, 21, [400, 200, 100], 8200, 0),      # the same where two 64-row tiles do not fit: 32-row tiles in turn
    (200, 33, [512, 512, 300], 130, 0),       # a head of two feature tiles; weights beyond 1 MB
    (200, 20, [512, 512, 300], 65600, 0),     # ... and 64-row tiles one per compute unit
    (211, 20, [512, 512, 256, 128], 4096, 0),       # the last size below the row-tile forward kernel
    (30, 5, [64] * 8, 100, 0),                # the most layers
    (211, 20, [512, 512, 256, 128], 12293, 0),      # row-tile forward kernel: rows gathered 16 at a time, ragged last ones
    (211, 20, [512, 512, 256, 128], 12293, 1),      # ... row by row (not 16-byte aligned)
    (211, 20, [512, 512, 256, 128], 4097, 1), (211, 20, [512, 512, 256, 128], 12287, 0),
    (211, 20, [512, 512, 512, 256], 4096, 0), (211, 20, [512, 512, 512, 256], 4097, 0),      # the same two kernels, widest shape
    (211, 20, [512, 512, 512, 256], 12287, 0), (211, 20, [512, 512, 512, 256], 12307, 0),
])
def test_agent_kernel_matches_the_per_layer_path(g, inst, obs, act, hidden, n, shift):
    """Both paths round the same activations to bf16 after sums in another order: an activation may land on the other
    neighbour (2^-8 of it), far less than 1e-2 of an output's norm; noise and log-density do not depend on them."""
    dev = torch.device("cuda:0")
    theta = torch.tensor(syn.make_model_params(obs, act, hidden, 5, policy_head_scale=0.5), device=dev)
    desc = g.model_desc(obs, act, list(hidden), g.dtype_code("bf16"), n)
    shadow = torch.zeros(g.gmi_model_shadow_bytes(desc), dtype=torch.uint8, device=dev)
    x = torch.randn(n * obs + shift, generator=torch.Generator().manual_seed(n)).to(dev)[shift:]
    torch.cuda.synchronize()
    model = g.gmi_model_bind(inst, desc, theta, shadow)
    g.gmi_model_refresh_shadow(inst, model)
    out = {}
    for fused in (1, 0):
        g.gmi_set_fusion(inst, fused)
        o = [torch.full(s, float("nan"), device=dev) for s in ((n, act), (n,), (n,), (n, act), (n,))]
        torch.cuda.synchronize()
        g.agent_act(inst, model, x, n, 42, 9, 100, *o[:4])
        g.agent_value(inst, model, x, n, o[4])
        g.gmi_sync(inst)
        out[fused] = [t.cpu().numpy() for t in o]
    g.gmi_set_fusion(inst, 1)
    g.gmi_model_destroy(model)
    for k in (0, 2, 3, 4):
        assert np.isfinite(out[1][k]).all()
        assert rel_l2(out[1][k], out[0][k]) <= 1e-2, k
    assert rel_l2(out[1][1], out[0][1]) <= 1e-6
    assert np.array_equal(out[1][2], out[1][4])      # agent_value is the same network pass


@pytest.mark.parametrize("obs,act,shift", [(211, 1, 0), (211, 3, 1), (193, 4, 0), (208, 7, 0), (208, 8, 1), (222, 9, 0), (223, 31, 3),
                                           (224, 32, 2)])
@pytest.mark.parametrize("hidden,n", [([512, 512, 256, 128], 769), ([512, 512, 512, 256], 832)])
def test_row_tile_decisions_match_the_per_layer_path(g, obs, act, hidden, n, shift):
    """Enough rows for 16 compute units to take the row-tile kernel: observation rows at every alignment and remainder, every
    remainder of the actions."""
    from paper_2206_08482_amd.instances import cu_masks
    masked = g.gmi_create(cu_masks(256, [16])[0])
    test_agent_kernel_matches_the_per_layer_path(g, masked, obs, act, hidden, n, shift)
    g.gmi_destroy(masked)


@pytest.mark.parametrize("obs,act,hidden,shift", [
    (108, 21, [400, 200, 100], 0), (107, 32, [400, 200, 100], 1), (97, 1, [200, 400, 100], 3), (110, 4, [200, 400, 100], 0),
    (57, 6, [256, 128, 64], 0), (62, 31, [256, 128, 64], 2), (23, 9, [256, 128, 64], 0), (5, 2, [256, 128, 64], 1)])
@pytest.mark.parametrize("n", [257, 321])
def test_row_tile_decisions_are_those_of_the_agent_kernel(g, inst, obs, act, hidden, n, shift):
    """The same rows on the whole device (the agent kernel) and on 16 compute units (enough rows for the row-tile kernel): bit for bit."""
    from paper_2206_08482_amd.instances import cu_masks
    dev = torch.device("cuda:0")
    masked = g.gmi_create(cu_masks(256, [16])[0])
    theta = torch.tensor(syn.make_model_params(obs, act, hidden, 5, policy_head_scale=0.5), device=dev)
    desc = g.model_desc(obs, act, list(hidden), g.dtype_code("bf16"), n)
    shadow = torch.zeros(g.gmi_model_shadow_bytes(desc), dtype=torch.uint8, device=dev)
    x = torch.randn(n * obs + shift, generator=torch.Generator().manual_seed(n)).to(dev)[shift:]
    torch.cuda.synchronize()
    out = []
    for h in (inst, masked):
        model = g.gmi_model_bind(h, desc, theta, shadow)
        g.gmi_model_refresh_shadow(h, model)
        o = [torch.full(s, float("nan"), device=dev) for s in ((n, act), (n,), (n,), (n, act), (n,))]
        torch.cuda.synchronize()
        g.agent_act(h, model, x, n, 42, 9, 100, *o[:4])
        g.agent_value(h, model, x, n, o[4])
        g.gmi_sync(h)
        out.append([t.cpu().numpy() for t in o])
        g.gmi_model_destroy(model)
    g.gmi_destroy(masked)
    for a, b in zip(*out):
        assert np.isfinite(a).all() and np.array_equal(a, b)


@pytest.mark.parametrize("obs,act,hidden,shift", [
    (108, 21, [400, 200, 100], 0), (66, 32, [400, 200, 100], 1), (127, 1, [200, 400, 100], 3), (211, 20, [512, 512, 256, 128], 0),
    (193, 7, [512, 512, 256, 128], 2), (256, 4, [512, 512, 512, 256], 1)])
@pytest.mark.parametrize("n", [513, 577])
def test_fp8_row_tile_decisions_are_those_of_the_agent_kernel(g, inst, obs, act, hidden, n, shift):
    """As above: more than 32 rows per compute unit."""
    from paper_2206_08482_amd.instances import cu_masks
    dev = torch.device("cuda:0")
    masked = g.gmi_create(cu_masks(256, [16])[0])
    theta = torch.tensor(syn.make_model_params(obs, act, hidden, 5, policy_head_scale=0.5), device=dev)
    x = torch.randn(n * obs + shift, generator=torch.Generator().manual_seed(n)).to(dev)[shift:]
    torch.cuda.synchronize()
    out = []
    for h in (inst, masked):
        w = g.gmi_fp8_bind(h, g.model_desc(obs, act, list(hidden), g.dtype_code("bf16"), n))
        g.gmi_fp8_refresh(h, w, theta)
        o = [torch.full(s, float("nan"), device=dev) for s in ((n, act), (n,), (n,), (n, act))]
        torch.cuda.synchronize()
        g.agent_act_fp8(h, w, x, n, 42, 9, 100, *o)
        g.gmi_sync(h)
        out.append([t.cpu().numpy() for t in o])
        g.gmi_fp8_destroy(w)
    g.gmi_destroy(masked)
    for a, b in zip(*out):
        assert np.isfinite(a).all() and np.array_equal(a, b)


@pytest.mark.parametrize("dtype,obs", [("bf16", 60), ("bf16", 48), ("bf16", 24), ("bf16", 4), ("fp8", 60), ("fp8", 23), ("fp8", 4)])
@pytest.mark.parametrize("act", [1, 8, 31])
@pytest.mark.parametrize("n", [1, 63, 65, 300])
def test_narrow_row_tile_decisions_are_those_of_the_agent_kernel(g, inst, dtype, obs, act, n):
    """256:128:64, which the row-tile kernel serves at every number of rows: against the same network on its first three observations
    alone, which the agent kernel serves (rows of fewer than four), the others being zero: products that add nothing.  Bit for bit."""
    hidden, dev = [256, 128, 64], torch.device("cuda:0")
    small = syn.make_model_params(3, act, hidden, 5, policy_head_scale=0.5)
    big, at = [], 0
    for out in (act, 1):
        prev = 3
        for i, w in enumerate(hidden + [out]):
            m = small[at:at + w * prev].reshape(w, prev)
            at += w * prev
            # the new columns repeat the first one: a layer's largest weight, and with it the fp8 scale, stays
            big += [np.concatenate([m, np.repeat(m[:, :1], obs - 3, 1)], 1).ravel() if i == 0 else m.ravel(), small[at:at + w]]
            at += w
            prev = w
    big = np.concatenate(big + [small[at:]]).astype(np.float32)
    x = torch.randn(n, 3, generator=torch.Generator().manual_seed(n)).to(dev)
    wide = torch.zeros(n, obs, device=dev)
    wide[:, :3] = x
    out = []
    for o, t, rows in ((3, small, x), (obs, big, wide)):
        theta = torch.tensor(t, device=dev)
        desc = g.model_desc(o, act, hidden, g.dtype_code("bf16"), n)
        r = [torch.full(s, float("nan"), device=dev) for s in ((n, act), (n,), (n,), (n, act))]
        shadow = torch.zeros(g.gmi_model_shadow_bytes(desc), dtype=torch.uint8, device=dev)
        torch.cuda.synchronize()
        if dtype == "fp8":
            model = g.gmi_fp8_bind(inst, desc)
            g.gmi_fp8_refresh(inst, model, theta)
            g.agent_act_fp8(inst, model, rows, n, 42, 9, 100, *r)
        else:
            model = g.gmi_model_bind(inst, desc, theta, shadow)
            g.gmi_model_refresh_shadow(inst, model)
            g.agent_act(inst, model, rows, n, 42, 9, 100, *r)
        g.gmi_sync(inst)
        (g.gmi_fp8_destroy if dtype == "fp8" else g.gmi_model_destroy)(model)
        out.append([v.cpu().numpy() for v in r])
    for a, b in zip(*out):
        assert np.isfinite(a).all() and np.array_equal(a, b)


@pytest.mark.parametrize("dtype", ["bf16", "fp8"])
@pytest.mark.parametrize("obs,act", [(60, 8), (24, 3), (23, 31)])
def test_narrow_row_tile_decisions_with_one_and_with_two_activation_areas(g, inst, dtype, obs, act):
    """A launch of at most one workgroup per compute unit takes its layers through two areas in turn, a larger one through one: the rows
    that both decide are the same bit for bit."""
    hidden, dev = [256, 128, 64], torch.device("cuda:0")
    few = 32 * torch.cuda.get_device_properties(0).multi_processor_count
    theta = torch.tensor(syn.make_model_params(obs, act, hidden, 5, policy_head_scale=0.5), device=dev)
    x = torch.randn(few + 1, obs, generator=torch.Generator().manual_seed(3)).to(dev)
    out = []
    for n in (few, few + 1):
        desc = g.model_desc(obs, act, hidden, g.dtype_code("bf16"), n)
        r = [torch.full(s, float("nan"), device=dev) for s in ((n, act), (n,), (n,), (n, act))]
        shadow = torch.zeros(g.gmi_model_shadow_bytes(desc), dtype=torch.uint8, device=dev)
        torch.cuda.synchronize()
        if dtype == "fp8":
            model = g.gmi_fp8_bind(inst, desc)
            g.gmi_fp8_refresh(inst, model, theta)
            g.agent_act_fp8(inst, model, x, n, 42, 9, 100, *r)
        else:
            model = g.gmi_model_bind(inst, desc, theta, shadow)
            g.gmi_model_refresh_shadow(inst, model)
            g.agent_act(inst, model, x, n, 42, 9, 100, *r)
        g.gmi_sync(inst)
        (g.gmi_fp8_destroy if dtype == "fp8" else g.gmi_model_destroy)(model)
        out.append([v.cpu().numpy() for v in r])
    for a, b in zip(*out):
        assert np.isfinite(b).all() and np.array_equal(a, b[:few])


@pytest.mark.parametrize("obs,act,hidden,n", [
    (211, 20, [512, 512, 256, 128], 32769),   # 128 rows on 16 waves
    (60, 8, [256, 128, 64], 32801),           # two 128-row tiles per compute unit
    (107, 21, [400, 200, 100], 8225),         # two 64-row tiles; rows of an odd length
    (45, 300, [100], 65),                     # a head of ten feature tiles
    (45, 510, [512, 512], 33),                # draws and densities do not fit beside the tile: a launch of their own
])
def test_fp8_agent_rows_do_not_depend_on_the_tile(g, inst, obs, act, hidden, n):
    """A row's results are the same whatever the workgroup's rows: a large batch against its rows in batches of 32, bit for
    bit (the small batches are compared with the oracle elsewhere)."""
    dev = torch.device("cuda:0")
    theta = torch.tensor(syn.make_model_params(obs, act, hidden, 5, policy_head_scale=0.5), device=dev)
    w = g.gmi_fp8_bind(inst, g.model_desc(obs, act, list(hidden), g.dtype_code("bf16"), n))
    x = torch.randn(n, obs, generator=torch.Generator().manual_seed(n)).to(dev)
    torch.cuda.synchronize()
    g.gmi_fp8_refresh(inst, w, theta)
    new = lambda k: [torch.full(s, float("nan"), device=dev) for s in ((k, act), (k,), (k,), (k, act))]
    big = new(n)
    torch.cuda.synchronize()
    g.agent_act_fp8(inst, w, x, n, 42, 9, 100, *big)
    for r0 in (0, 32 * (n // 64), 32 * ((n - 1) // 32)):
        k = min(32, n - r0)
        o, xs = new(k), x[r0:r0 + k].clone()
        torch.cuda.synchronize()
        g.agent_act_fp8(inst, w, xs, k, 42, 9, 100 + r0, *o)
        g.gmi_sync(inst)
        for a, b in zip(big, o):
            assert torch.isfinite(b).all()
            assert torch.equal(a[r0:r0 + k], b)
    g.gmi_fp8_destroy(w)


@pytest.mark.parametrize("obs,act,hidden,n,T", [
    (5, 1, [32], 1, 2),                       # one env, rows of an odd length
    (45, 12, [128, 128], 33, 3),              # a ragged second tile; slots that are not 16-byte aligned
    (107, 21, [400, 200, 100], 600, 3),       # 16 envs per workgroup, two envs per simulator item
    (45, 12, [100], 16400, 2),                # 64 envs per workgroup
])
def test_streamed_collection_equals_the_step_by_step_calls(g, obs, act, hidden, n, T):
    """Models whose weights the one-launch collection streams (the policy net in the launch, the values afterwards): every
    array bit for bit that of agent_act / env_step / collect_experience, over two iterations in a row."""
    from paper_2206_08482_amd.runner import PPOSession
    rng = np.random.default_rng(9)
    theta = syn.make_model_params(obs, act, hidden, 5, policy_head_scale=0.5)
    a_mat = (0.9 * np.eye(obs) + 0.01 * rng.standard_normal((obs, obs))).astype(np.float32)
    b_mat = (0.1 * rng.standard_normal((obs, act))).astype(np.float32)
    state0 = rng.standard_normal((n, obs)).astype(np.float32)
    ses = [PPOSession(n_envs=n, obs_dim=obs, act_dim=act, hidden=hidden, horizon=T, dtype="bf16", theta=theta, a_mat=a_mat,
                      b_mat=b_mat, state0=state0, noise_std=0.01, reward_scale=1.0, done_period=0, done_threshold=(1 << 32) // 5,
                      seed=11, minibatch=n, fused_rollout=f) for f in (True, False)]
    for it in range(2):
        for s in ses:
            s.rollout(it)
            s.sync()
        assert ses[0].fused_rollout
        ga, gb = (s.buf.to_numpy() for s in ses)
        for k in ("obs", "act", "logp", "val", "rew", "done"):
            assert np.array_equal(ga[k], gb[k]), (it, k)
        assert np.array_equal(ses[0].state().cpu().numpy(), ses[1].state().cpu().numpy())
        assert np.array_equal(ses[0].last_value.cpu().numpy(), ses[1].last_value.cpu().numpy())
    for s in ses:
        s.close()


@pytest.mark.parametrize("dtype,fused", [("bf16", 1), ("bf16", 0), ("f32", 1), ("f32", 0)])
def test_probability_ratio_is_the_accurate_exponential(g, inst, dtype, fused):
    """The ratio of a model without a compiled trainer kernel is expf of the log-density difference, also far from 1.  All
    policy weights are zero and the action is the mean, so the log-density is -log(2 pi) / 2 exactly; one sample per call,
    and an advantage whose sign keeps the unclipped term: the policy loss is the ratio itself.  Bound: the difference is
    one fp32 subtraction on both sides, expf is within 1 ulp (1.2e-7), so 4e-7; a 2^x of an fp32 product x log2 e is off by
    up to |x| 2^-24 (1.4e-6 was measured at 37.7)."""
    obs, act, hidden, N = 5, 1, (32,), 12
    model, buf, keep = _setup(g, inst, obs, act, hidden, dtype, 1, N, N)
    theta, shadow, m, v, rb = keep
    theta.zero_()
    x = np.array([0.0, 0.3, -0.7, 2.5, -3.3, 7.9, -9.1, 13.7, 21.3, -25.9, 37.7, 43.1], np.float32)
    lp = np.float32(-0.918938533204672742)
    logp = (lp - x).astype(np.float32)
    rb.act.zero_()
    rb.logp.copy_(torch.tensor(logp)[None])
    rb.adv.copy_(torch.tensor(np.where(x > 0, -1, 1).astype(np.float32))[None])
    torch.cuda.synchronize()
    g.gmi_model_refresh_shadow(inst, model)
    g.gmi_set_fusion(inst, fused)
    hp = g.ppo_hparams(clip=0.2, c_v=0.5, c_e=0.0, minibatch=1)
    grad = torch.zeros(theta.numel(), device="cuda:0")
    stats = torch.zeros(N, 5, device="cuda:0")
    idx = torch.arange(N, dtype=torch.int32, device="cuda:0")
    torch.cuda.synchronize()
    for i in range(N):
        g.ppo_gradient(inst, model, buf, hp, idx[i:], 1, grad, stats[i])
    g.gmi_sync(inst)
    g.gmi_set_fusion(inst, 1)
    got = np.abs(stats[:, 0].cpu().numpy().astype(np.float64))
    want = np.exp((lp - logp).astype(np.float32).astype(np.float64))
    assert np.abs(got / want - 1).max() <= 4e-7, np.abs(got / want - 1)
    g.gmi_buffer_destroy(buf)
    g.gmi_model_destroy(model)


@pytest.mark.parametrize("obs,hidden", [(60, (256, 128, 64)), (23, (256, 128, 64)), (108, (400, 200, 100)), (108, (200, 400, 100)),
                                        (211, (512, 512, 256, 128)), (211, (512, 512, 512, 256))])
def test_probability_ratio_of_the_row_tile_kernel(g, inst, obs, hidden):
    """As above, for every shape with a compiled trainer kernel: the policy loss is the ratio, the gradient of log_std (a mean at
    the action: g (0 - 1) with g = -ratio advantage) the ratio times the advantage, both to 4e-7.  The class's stated work says
    that the row-tile kernel ran."""
    act, N = 1, 12
    model, buf, keep = _setup(g, inst, obs, act, hidden, "bf16", 1, N, N)
    theta, shadow, m, v, rb = keep
    theta.zero_()
    x = np.array([0.0, 0.3, -0.7, 2.5, -3.3, 7.9, -9.1, 13.7, 21.3, -25.9, 37.7, 43.1], np.float32)
    lp = np.float32(-0.918938533204672742)
    logp = (lp - x).astype(np.float32)
    adv = np.where(x > 0, -1, 1).astype(np.float32)
    rb.act.zero_()
    rb.logp.copy_(torch.tensor(logp)[None])
    rb.adv.copy_(torch.tensor(adv)[None])
    torch.cuda.synchronize()
    g.gmi_model_refresh_shadow(inst, model)
    hp = g.ppo_hparams(clip=0.2, c_v=0.5, c_e=0.0, minibatch=1)
    grad = torch.zeros(N, theta.numel(), device="cuda:0")
    stats = torch.zeros(N, 5, device="cuda:0")
    idx = torch.arange(N, dtype=torch.int32, device="cuda:0")
    torch.cuda.synchronize()
    cls = [g.gmi_profile_class_name(c) for c in range(g.gmi_profile_classes())].index("chain_train")
    g.gmi_profile_enable(inst, 1 << cls)
    for i in range(N):
        g.ppo_gradient(inst, model, buf, hp, idx[i:], 1, grad[i], stats[i])
    g.gmi_sync(inst)
    assert g.gmi_profile_read(inst, cls)[1] == N and g.gmi_profile_work(inst, cls)[0] > 0
    g.gmi_profile_enable(inst, 0)
    want = np.exp((lp - logp).astype(np.float32).astype(np.float64))
    for got in (-stats[:, 0].cpu().numpy(), grad[:, -1].cpu().numpy()):
        assert np.abs(got * adv / want - 1).max() <= 4e-7, np.abs(got * adv / want - 1)
    g.gmi_buffer_destroy(buf)
    g.gmi_model_destroy(model)


def _collecting_sessions(obs, act, hidden, dtype, n, T, cus, seed=9):
    """The same session with the one-launch collection and with the step-by-step calls, on `cus` compute units (None: all)."""
    from paper_2206_08482_amd.instances import cu_masks
    from paper_2206_08482_amd.runner import PPOSession
    rng = np.random.default_rng(seed)
    theta = syn.make_model_params(obs, act, hidden, 5, policy_head_scale=0.5)
    a_mat = (0.9 * np.eye(obs) + 0.01 * rng.standard_normal((obs, obs))).astype(np.float32)
    b_mat = (0.1 * rng.standard_normal((obs, act))).astype(np.float32)
    state0 = rng.standard_normal((n, obs)).astype(np.float32)
    mask = cu_masks(256, [cus])[0] if cus else None
    return [PPOSession(n_envs=n, obs_dim=obs, act_dim=act, hidden=hidden, horizon=T, dtype=dtype, theta=theta, a_mat=a_mat,
                       b_mat=b_mat, state0=state0, noise_std=0.01, reward_scale=1.0, done_period=0, cu_mask=mask,
                       done_threshold=(1 << 32) // 5, seed=11, minibatch=n, fused_rollout=f) for f in (True, False)]


@pytest.mark.parametrize("obs,act,hidden,n,T,cus", [
    (1, 1, [32], 1, 2, None),                  # one env
    (17, 6, [64, 64], 33, 3, None),            # weights in LDS, a ragged third tile of 16
    (45, 12, [128, 128], 100, 3, None),        # weights that do not fit LDS
    (17, 6, [64, 64], 4113, 2, None),          # the first tiles of 32 envs
    (17, 6, [64, 64], 8211, 2, None),          # 32 envs per workgroup, 257 tiles: one workgroup takes two
    (45, 12, [128, 128], 8211, 2, None),
    (17, 6, [64, 64], 300, 3, 8),              # ten tiles of 32 on eight compute units
    (45, 12, [128, 128], 300, 3, 8),
    (200, 20, [256, 256], 200, 2, 8),          # 32 envs do not fit: thirteen tiles of 16 on eight
])
def test_fp32_collection_equals_the_step_by_step_calls(g, obs, act, hidden, n, T, cus):
    """Both are fp32 arithmetic with sums in orders of their own: 1e-5 as everywhere on this path; done flags exactly."""
    ses = _collecting_sessions(obs, act, hidden, "f32", n, T, cus)
    for it in range(2):
        for s in ses:
            s.rollout(it)
            s.sync()
        assert ses[0].fused_rollout_f32 and not ses[1].fused_rollout_f32
        ga, gb = (s.buf.to_numpy() for s in ses)
        assert np.array_equal(ga["done"], gb["done"])
        for k in ("obs", "act", "logp", "val", "rew"):
            assert rel_l2(ga[k], gb[k]) <= 1e-5, (it, k, rel_l2(ga[k], gb[k]))
        assert rel_l2(ses[0].state().cpu().numpy(), ses[1].state().cpu().numpy()) <= 1e-5
        assert rel_l2(ses[0].last_value.cpu().numpy(), ses[1].last_value.cpu().numpy()) <= 1e-5
        assert torch.equal(ses[0].episode_step, ses[1].episode_step)
    for s in reversed(ses):
        s.close()


@pytest.mark.parametrize("obs,act,hidden,n,shift", [
    (8, 2, [32, 32], 4093, 0), (8, 2, [32, 32], 8195, 1),                 # 32 and 64 rows, weights in LDS
    (60, 8, [256, 128, 64], 4099, 1), (60, 8, [256, 128, 64], 8193, 0),   # ... and streamed
    (45, 12, [128, 128], 1, 0), (45, 33, [128, 100], 17, 0),              # 16 rows; a head of three feature tiles
    (108, 21, [256, 128], 8200, 0), (200, 20, [512, 512], 8200, 0),       # 64 rows do not fit; 32 do not either
])
def test_fp32_agent_matches_the_per_layer_path(g, inst, obs, act, hidden, n, shift):
    dev = torch.device("cuda:0")
    theta = torch.tensor(syn.make_model_params(obs, act, hidden, 5, policy_head_scale=0.5), device=dev)
    x = torch.randn(n * obs + shift, generator=torch.Generator().manual_seed(n)).to(dev)[shift:]
    torch.cuda.synchronize()
    model = g.gmi_model_bind(inst, g.model_desc(obs, act, list(hidden), g.dtype_code("f32"), n), theta, None)
    out = {}
    for fused in (1, 0):
        g.gmi_set_fusion(inst, fused)
        o = [torch.full(s, float("nan"), device=dev) for s in ((n, act), (n,), (n,), (n, act), (n,))]
        torch.cuda.synchronize()
        g.agent_act(inst, model, x, n, 42, 9, 100, *o[:4])
        g.agent_value(inst, model, x, n, o[4])
        g.gmi_sync(inst)
        out[fused] = [t.cpu().numpy() for t in o]
    g.gmi_set_fusion(inst, 1)
    g.gmi_model_destroy(model)
    for k in range(5):
        assert np.isfinite(out[1][k]).all()
        assert rel_l2(out[1][k], out[0][k]) <= 1e-5, (k, rel_l2(out[1][k], out[0][k]))
        row = np.abs(out[1][k] - out[0][k]).reshape(n, -1).max(axis=1)      # every row on its own
        assert row.max() <= 1e-4 * np.abs(out[0][k]).max(), (k, int(row.argmax()))


@pytest.mark.parametrize("obs,act,hidden,n,T", [
    (45, 12, [128, 128], 600, 3),              # values: 128 rows per workgroup, 20 items on eight compute units
    (107, 21, [400, 200, 100], 600, 3),        # 32 rows, 76 items
    (60, 8, [256, 256], 161, 1),               # the last value alone beside one step
])
def test_values_of_a_collection_on_few_compute_units(g, obs, act, hidden, n, T):
    """The values of all slots come from workgroups that the instance's compute units hold, each taking several items:
    bit for bit those of the step-by-step calls."""
    ses = _collecting_sessions(obs, act, hidden, "bf16", n, T, 8)
    for it in range(2):
        for s in ses:
            s.rollout(it)
            s.sync()
        assert ses[0].fused_rollout and not ses[1].fused_rollout
        ga, gb = (s.buf.to_numpy() for s in ses)
        for k in ("obs", "act", "logp", "val", "rew", "done"):
            assert np.array_equal(ga[k], gb[k]), (it, k)
        assert torch.equal(ses[0].last_value, ses[1].last_value)
    for s in reversed(ses):
        s.close()


@pytest.mark.parametrize("n,cus,tile", [(12341, None, True), (4097, None, True), (4096, None, False), (777, 16, True), (257, 16, True),
                                        (256, 16, False)])
@pytest.mark.parametrize("hidden", [[512, 512, 256, 128], [512, 512, 512, 256]])
def test_two_launch_collection_through_the_row_tile_kernel(g, hidden, n, cus, tile):
    """Beyond 16 envs per compute unit (4096 on the whole device) the 512-wide models collect through the forward-only
    row-tile kernel, as agent_act does: bit for bit the step-by-step calls, a ragged last tile included.  Of the class's
    kernels only that one states its work."""
    ses = _collecting_sessions(211, 20, hidden, "bf16", n, 2, cus)
    cls = [g.gmi_profile_class_name(c) for c in range(g.gmi_profile_classes())].index("fused_agent")
    for it in range(2):
        for s in ses:
            g.gmi_profile_enable(s.gmi, 1 << cls)
            s.rollout(it)
            s.sync()
            assert (g.gmi_profile_work(s.gmi, cls)[0] > 0) == tile
            g.gmi_profile_enable(s.gmi, 0)
        assert ses[0].fused_rollout and not ses[1].fused_rollout
        ga, gb = (s.buf.to_numpy() for s in ses)
        for k in ("obs", "act", "logp", "val", "rew", "done"):
            assert np.array_equal(ga[k], gb[k]), (it, k)
        assert torch.equal(ses[0].state(), ses[1].state()) and torch.equal(ses[0].last_value, ses[1].last_value)
    for s in reversed(ses):
        s.close()


@pytest.mark.parametrize("obs,n", [(1, 4096), (2, 33), (3, 700), (5, 17)])
def test_fp32_elu_is_within_an_ulp(g, inst, obs, n):
    """One hidden unit copies the last observation, the head copies the unit: the mean is ELU(x) itself (every other product is
    zero).  The kernel's e^x - 1 is within 0.86 ulp of the exact value, its place in a sum of zeros exact: 1 ulp; beyond -30 and
    at -inf it is -1."""
    act, hidden, dev = 2, [33], torch.device("cuda:0")
    theta = torch.zeros(sum(33 * (obs + 1) + 33 * o + o for o in (act, 1)) + act)
    theta[obs - 1] = 1.0                          # policy W0[0][obs - 1]
    theta[33 * (obs + 1)] = 1.0                   # policy W1[0][0]
    rng = np.random.default_rng(obs)
    x = rng.standard_normal((n, obs)).astype(np.float32)
    x[:, -1] = np.concatenate([-np.exp(rng.uniform(-20, 3.4, n - 4)), [-31.0, -1e30, -0.0, 2.5]]).astype(np.float32)
    xd, theta = torch.tensor(x, device=dev), theta.to(dev)
    model = g.gmi_model_bind(inst, g.model_desc(obs, act, hidden, g.dtype_code("f32"), n), theta, None)
    o = [torch.zeros(s, device=dev) for s in ((n, act), (n,), (n,), (n, act))]
    torch.cuda.synchronize()
    g.agent_act(inst, model, xd, n, 42, 9, 0, *o)
    g.gmi_sync(inst)
    g.gmi_model_destroy(model)
    got = o[3].cpu().numpy()[:, 0].astype(np.float64)
    z = x[:, -1].astype(np.float64)
    want = np.where(z > 0, z, np.expm1(np.minimum(z, 0.0)))
    ulp = np.spacing(np.abs(want).astype(np.float32)).astype(np.float64)
    assert (np.abs(got - want) <= ulp).all(), (np.abs(got - want) / ulp).max()


@pytest.mark.parametrize("obs,act,hidden,n,T", [
    (1, 1, [32], 1, 3), (2, 1, [33, 65], 15, 4), (7, 3, [48], 16, 3),      # 16 envs; 1, 2 and 3 products left over of a group of four
    (3, 21, [40], 17, 3),                      # more blocks of actions than of states
    (45, 12, [128, 128], 100, 5), (130, 9, [300, 100], 33, 3),      # two weight rounds per layer, nine state tiles
    (254, 24, [256], 40, 3),                   # the simulator's matrix read from memory
    (90, 6, [512, 100], 17000, 2),             # 32 envs, the matrix staged at every step
    (200, 30, [64], 16500, 2),                 # two states of 64 envs do not fit: 32
    (120, 6, [64, 100], 17000, 2),             # 64 envs, a step's draws ahead of it
    (300, 16, [32], 20000, 2),                 # 32 envs, the same
])
def test_collection_at_the_edges_of_its_layouts(g, obs, act, hidden, n, T):
    """Same draws, same sums in the same order: bit for bit the step-by-step calls."""
    ses = _collecting_sessions(obs, act, hidden, "bf16", n, T, None)
    for it in range(2):
        for s in ses:
            s.rollout(it)
            s.sync()
        assert ses[0].fused_rollout and not ses[1].fused_rollout
        ga, gb = (s.buf.to_numpy() for s in ses)
        for k in ("obs", "act", "logp", "val", "rew", "done"):
            assert np.array_equal(ga[k], gb[k]), (it, k)
        assert torch.equal(ses[0].state(), ses[1].state()) and torch.equal(ses[0].last_value, ses[1].last_value)
        assert torch.equal(ses[0].episode_step, ses[1].episode_step)
    for s in reversed(ses):
        s.close()


@pytest.mark.parametrize("obs,act,hidden,n", [(408, 40, [32], 40), (380, 9, [32], 20), (3, 21, [40], 17)])
def test_fp32_collection_at_the_edges_of_its_layout(g, obs, act, hidden, n):
    """A step's draws ahead of it (408:32:40), the matrix from memory; 1e-5 as everywhere on this path."""
    ses = _collecting_sessions(obs, act, hidden, "f32", n, 3, None)
    for s in ses:
        s.rollout(0)
        s.sync()
    assert ses[0].fused_rollout_f32 and not ses[1].fused_rollout_f32
    ga, gb = (s.buf.to_numpy() for s in ses)
    assert np.array_equal(ga["done"], gb["done"])
    for k in ("obs", "act", "logp", "val", "rew"):
        assert rel_l2(ga[k], gb[k]) <= 1e-5, (k, rel_l2(ga[k], gb[k]))
    for s in reversed(ses):
        s.close()


@pytest.mark.parametrize("obs,act,hidden,n,T,cus", [
    (64, 1, [64], 16, 4, None),                # two layers; the widest input in registers, whole tiles
    (65, 7, [17, 64], 33, 3, None),            # the first layer's weights in LDS; a ragged third tile
    (3, 24, [64, 33, 16], 70, 3, 8),           # more blocks of actions than of states; two heads' tiles; one workgroup per tile
    (130, 9, [16, 16], 40, 3, None),           # nine state tiles: a simulator wave has three
    (256, 24, [16], 18, 2, None),              # the simulator's matrix in memory
    (128, 4, [64], 21, 3, None),               # so too, its rows without padding, one product behind the state's: the last one
    (6, 2, [64, 64], 300, 5, 8),               # nineteen tiles on eight compute units; two products behind the state's
])
def test_fp32_collection_with_the_roles_on_waves_of_their_own(g, obs, act, hidden, n, T, cus):
    """Small nets (layers of at most 64 units).  1e-5 as everywhere on this path; done flags and counters exactly."""
    ses = _collecting_sessions(obs, act, hidden, "f32", n, T, cus)
    for it in range(2):
        for s in ses:
            s.rollout(it)
            s.sync()
        assert ses[0].fused_rollout_f32 and not ses[1].fused_rollout_f32
        ga, gb = (s.buf.to_numpy() for s in ses)
        assert np.array_equal(ga["done"], gb["done"]) and ga["done"].any()
        for k in ("obs", "act", "logp", "val", "rew"):
            assert rel_l2(ga[k], gb[k]) <= 1e-5, (it, k, rel_l2(ga[k], gb[k]))
        assert rel_l2(ses[0].state().cpu().numpy(), ses[1].state().cpu().numpy()) <= 1e-5
        assert rel_l2(ses[0].last_value.cpu().numpy(), ses[1].last_value.cpu().numpy()) <= 1e-5
        assert torch.equal(ses[0].episode_step, ses[1].episode_step)
    for s in reversed(ses):
        s.close()


@pytest.mark.parametrize("obs,act,hidden,fused", [
    (60, 8, (256, 128, 64), 1), (108, 21, (400, 200, 100), 1), (211, 20, (512, 512, 256, 128), 1), (108, 21, (400, 200, 100), 0),
    (17, 40, (800, 300), 0), (3, 1, (32,), 0), (300, 5, (1100, 1100, 64), 0)])
def test_weight_gradient_splits_sum_to_the_gradient_of_the_pieces(g, inst, obs, act, hidden, fused):
    """The rows of a weight gradient are split among more or fewer workgroups layer by layer, tiles of a side are of equal size, and layers
    that the two nets do not share (a policy head wider than 32) have workgroups of their own.  Against the mean of 64-row pieces, which are
    not split: the gradient at the loss scales by a power of two, so every bf16 value is the same and only the order of the fp32 sums
    differs (2048 terms: well within 1e-4 of a tensor's norm); and against the fp32 kernels at the bf16 band, per tensor."""
    rows, piece = 2048, 64
    hp = lambda n: g.ppo_hparams(clip=1e3, c_v=0.5, c_e=0.0, minibatch=n)      # no sample at a clip boundary
    got = {}
    for dtype in ("bf16", "f32"):
        model, buf, keep = _setup(g, inst, obs, act, hidden, dtype, 2, rows // 2, rows)
        n = keep[0].numel()
        idx = torch.tensor(np.random.default_rng(1).permutation(rows).astype(np.int32), device="cuda:0")
        grad, part, stats = torch.zeros(n, device="cuda:0"), torch.zeros(rows // piece, n, device="cuda:0"), torch.zeros(5, device="cuda:0")
        torch.cuda.synchronize()
        g.gmi_set_fusion(inst, fused)
        g.ppo_gradient(inst, model, buf, hp(rows), idx, rows, grad, stats)
        if dtype == "bf16":
            for k in range(rows // piece):
                g.ppo_gradient(inst, model, buf, hp(piece), idx[k * piece:(k + 1) * piece], piece, part[k], stats)
        g.gmi_sync(inst)
        g.gmi_set_fusion(inst, 1)
        got[dtype] = grad.cpu().numpy()
        if dtype == "bf16":
            got["pieces"] = part.double().mean(0).cpu().numpy()
        g.gmi_buffer_destroy(buf)
        g.gmi_model_destroy(model)
    off = 0
    for out_dim in (act, 1):
        prev = obs
        for o in (*hidden, out_dim):
            for n_el in (prev * o, o):
                s = slice(off, off + n_el)
                assert rel_l2(got["bf16"][s], got["pieces"][s]) <= 1e-4, (off, rel_l2(got["bf16"][s], got["pieces"][s]))
                assert rel_l2(got["bf16"][s], got["f32"][s]) <= 2e-2, (off, rel_l2(got["bf16"][s], got["f32"][s]))
                off += n_el
            prev = o
