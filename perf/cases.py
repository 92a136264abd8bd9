"""What a user of this framework has it do, as cases to be timed.

Three kinds of pass, all through the public entry points:

  train     one synchronized PPO iteration of one instance (runner.PPOSession): reset of the environments, collection
            of a horizon of experience, GAE, and the epochs of minibatch updates -- forward, loss, backward, Adam
  serve     one action decision of an agent that only serves: agent_act (fp32, bf16) or agent_act_fp8
  pipeline  one iteration of several agent instances that feed one trainer instance on the same GPU
            (instances.InstancePipeline: agents on disjoint sets of compute units, hand-offs ordered by the host)

Models, environments and hyper-parameters: the configurations of workloads/synthetic.py (the benchmark's C1 .. C5 and
the policy models of the paper's Table 6), and multilayer perceptrons of arbitrary width as a user's own task has them.
"""
import math

import numpy as np
import torch

import paper_2206_08482_amd as gmi
from paper_2206_08482_amd.instances import InstancePipeline, cu_masks
from paper_2206_08482_amd.runner import PPOSession

GAMMA, LAM = 0.99, 0.95
HYPER = dict(clip=0.2, c_v=0.5, c_e=0.0, lr=3e-4, beta1=0.9, beta2=0.999, adam_eps=1e-8)

# obs, act, hidden widths, reward scale of the configurations' bf16 models
MODELS = {
    "C2": (60, 8, "256-128-64", 1.0),
    "C3": (108, 21, "400-200-100", 1.0),
    "C4": (211, 20, "512-512-256-128", 0.01),
    "AY": (48, 12, "256-128-64", 1.0),
    "BB": (24, 3, "256-128-64", 1.0),
    "FC": (23, 9, "256-128-64", 1.0),
    "HM": (108, 21, "200-400-100", 1.0),
    "SH": (211, 20, "512-512-512-256", 0.01),
}
WIDTHS = (32, 48, 64, 100, 128, 192, 200, 256, 300, 400, 512)


def train(obs, act, hidden, dtype, envs, horizon, epochs, minibatch, reward_scale=1.0, done_period=0):
    return dict(kind="train", obs=obs, act=act, hidden=hidden, dtype=dtype, envs=envs, horizon=horizon, epochs=epochs,
                minibatch=minibatch, reward_scale=reward_scale, done_period=done_period)


def serve(obs, act, hidden, dtype, rows):
    return dict(kind="serve", obs=obs, act=act, hidden=hidden, dtype=dtype, rows=rows)


def pipeline(obs, act, hidden, agents, envs, horizon, epochs, minibatch, reward_scale=1.0):
    return dict(kind="pipeline", obs=obs, act=act, hidden=hidden, dtype="bf16", agents=agents, envs=envs, horizon=horizon,
                epochs=epochs, minibatch=minibatch, reward_scale=reward_scale, done_period=0)


def listed():
    o2, a2, h2, _ = MODELS["C2"]
    o3, a3, h3, _ = MODELS["C3"]
    o4, a4, h4, r4 = MODELS["C4"]
    return [
        # the smallest training run (configuration C1): 64 environments, fp32, every launch is latency
        dict(train(8, 2, "32-32", "f32", 64, 16, 1, 256, done_period=16), name="train C1 f32"),
        # a user's own small task in full precision: classic-control / locomotion sizes, two layers of 64
        dict(train(17, 6, "64-64", "f32", 512, 32, 4, 4096), name="train 17:64:64:6 f32"),
        # configuration C2, the Ant-sized model: the ordinary training run
        dict(train(o2, a2, h2, "bf16", 4096, 16, 4, 32768), name="train C2"),
        # configuration C3, the Humanoid-sized model with a longer horizon
        dict(train(o3, a3, h3, "bf16", 4096, 32, 5, 32768), name="train C3"),
        # configuration C4, the largest model and batch
        dict(train(o4, a4, h4, "bf16", 16384, 16, 5, 32768, r4), name="train C4"),
        # a user's own model and odd sizes: 1000 environments, 24 steps, minibatches of 6000
        dict(train(45, 12, "128-128", "bf16", 1000, 24, 4, 6000), name="train 45:128:128:12"),
        # configuration C5: four agent instances and a trainer instance share the GPU
        dict(pipeline(o3, a3, h3, 4, 4096, 32, 5, 65536), name="pipeline C5"),
        # one environment asks for one action: the latency of a call
        dict(serve(o2, a2, h2, "bf16", 1), name="serve C2 x1"),
        # agents of the configurations at their environment counts, and one count that fills no tile
        dict(serve(o3, a3, h3, "bf16", 5000), name="serve C3 x5000"),
        dict(serve(o4, a4, h4, "bf16", 16384), name="serve C4 x16384"),
        # the same in fp8, for a large fleet
        dict(serve(o4, a4, h4, "fp8", 65536), name="serve C4 fp8 x65536"),
        # full-precision serving of a moderate fleet
        dict(serve(o2, a2, h2, "f32", 2048), name="serve C2 f32 x2048"),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _own_model(rng, widest, layers):
    """A user's own model: one to `layers` hidden layers that do not widen towards the head."""
    ws = sorted((rng.choice([w for w in WIDTHS if w <= widest]) for _ in range(rng.randint(1, layers))), reverse=True)
    return _log(rng, 4, 256), rng.randint(1, 24), "-".join(str(w) for w in ws), 0.1


def _model(rng, dtype):
    if dtype == "f32":
        return _own_model(rng, 256, 3)
    return MODELS[rng.choice(sorted(MODELS))] if rng.random() < 0.6 else _own_model(rng, 512, 4)


def draw(rng):
    u = rng.random()
    if u < 0.08:
        o, a, h, r = MODELS[rng.choice(("C2", "C3", "AY", "FC", "HM"))]
        agents, envs, horizon = rng.choice((2, 4)), 8 * _log(rng, 32, 512), rng.choice((8, 16, 32))
        return pipeline(o, a, h, agents, envs, horizon, rng.randint(1, 5), agents * envs * horizon // rng.choice((4, 8)), r)
    if u < 0.55:
        dtype = "f32" if rng.random() < 0.25 else "bf16"
        o, a, h, r = _model(rng, dtype)
        horizon, epochs, envs = rng.randint(8, 32), rng.randint(1, 5), _log(rng, 32, 16384)
        most = 6e9 if dtype == "f32" else 2.5e12      # a third of C4's products; the fp32 path runs at vector rates
        while True:
            batch = envs * horizon
            parts = [k for k in (1, 2, 3, 4, 5, 6, 8) if batch % k == 0 and batch // k <= 65536]
            if parts:
                c = train(o, a, h, dtype, envs, horizon, epochs, batch // rng.choice(parts), r)
                if work(c)["flops"] <= most:
                    return c
            envs = max(8, envs * 3 // 4)
    dtype = rng.choice(("bf16", "bf16", "fp8", "f32"))
    o, a, h, _ = _model(rng, dtype)
    rows = _log(rng, 1, 262144)
    while dtype == "f32" and work(serve(o, a, h, dtype, rows))["flops"] > 3e9:
        rows //= 2
    return serve(o, a, h, dtype, rows)


# ------------------------------------------------------------------------------------------------ inputs
def _widths(case):
    return [int(w) for w in case["hidden"].split("-")]


def _theta(case, rng):
    """Flat parameter vector as a trainer initialises it: W ~ N(0, 1 / fan_in), small biases, the policy head scaled."""
    parts = []
    for out, head in ((case["act"], 0.01), (1, 1.0)):
        prev, dims = case["obs"], _widths(case) + [out]
        for i, n in enumerate(dims):
            s = head if i == len(dims) - 1 else 1.0
            parts.append(s / math.sqrt(prev) * rng.standard_normal(n * prev, dtype=np.float32))
            parts.append(0.01 * s * rng.standard_normal(n, dtype=np.float32))
            prev = n
    parts.append(np.zeros(case["act"], np.float32))
    return np.concatenate(parts).astype(np.float32)


def _env(case, rng):
    """Dynamics of the synthetic environment: A = 0.95 I + 0.01 N(0, 1), B = 0.1 N(0, 1)."""
    o, a = case["obs"], case["act"]
    a_mat = 0.95 * np.eye(o, dtype=np.float32) + 0.01 * rng.standard_normal((o, o), dtype=np.float32)
    return a_mat, 0.1 * rng.standard_normal((o, a), dtype=np.float32)


_instance = []


def _one_instance():
    """The unmasked instance that training and serving passes run on: a program keeps one for its lifetime, and its passes
    follow one another on that instance's stream."""
    if not _instance:
        _instance.append(gmi.gmi_create())
    return _instance[0]


class _Train:
    def __init__(self, case, seed):
        rng = np.random.default_rng(seed)
        a_mat, b_mat = _env(case, rng)
        state0 = rng.standard_normal((case["envs"], case["obs"]), dtype=np.float32)
        self.case = case
        self.ses = PPOSession(n_envs=case["envs"], obs_dim=case["obs"], act_dim=case["act"], hidden=_widths(case),
                              horizon=case["horizon"], dtype=case["dtype"], theta=_theta(case, rng), a_mat=a_mat,
                              b_mat=b_mat, state0=state0, noise_std=0.01, reward_scale=case["reward_scale"],
                              done_period=case["done_period"],
                              done_threshold=0 if case["done_period"] else (1 << 32) // 1000, seed=seed,
                              minibatch=case["minibatch"], gmi=_one_instance())
        self.state0 = torch.tensor(state0, device="cuda:0")
        self.no_steps = torch.zeros_like(self.ses.episode_step)
        updates = case["epochs"] * (case["envs"] * case["horizon"] // case["minibatch"])
        self.stats = torch.zeros(updates, 5, device="cuda:0")
        gmi.gmi_wait_stream(self.ses.gmi)
        self.iteration = 0

    def step(self):
        s, c = self.ses, self.case
        # fresh environments: the synthetic dynamics grow over long horizons
        gmi.gmi_transfer(s.gmi, s.gmi, self.state0, s.obs[s.cur], self.state0.numel() * 4)
        gmi.gmi_transfer(s.gmi, s.gmi, self.no_steps, s.episode_step, self.no_steps.numel() * 4)
        s.rollout(self.iteration)
        s.gae(GAMMA, LAM, True)
        s.update(self.iteration, epochs=c["epochs"], minibatch=c["minibatch"], stats=self.stats, **HYPER)
        self.iteration += 1
        b = s.buf
        return dict(theta=s.theta, adam_m=s.adam_m, adam_v=s.adam_v, stats=self.stats, obs=b.obs, act=b.act, logp=b.logp,
                    val=b.val, rew=b.rew, done=b.done, adv=b.adv, ret=b.ret, last_value=s.last_value, state=s.state(),
                    episode_step=s.episode_step)

    def __del__(self):
        if hasattr(self, "ses"):
            self.ses.close()


class _Serve:
    def __init__(self, case, seed):
        rng = np.random.default_rng(seed)
        n, dev = case["rows"], "cuda:0"
        self.n, self.seed, self.calls, self.fp8 = n, seed, 0, case["dtype"] == "fp8"
        self.theta = torch.tensor(_theta(case, rng), device=dev)
        self.obs = torch.tensor(rng.standard_normal((n, case["obs"]), dtype=np.float32), device=dev)
        self.act = torch.zeros(n, case["act"], device=dev)
        self.mu = torch.zeros(n, case["act"], device=dev)
        self.logp = torch.zeros(n, device=dev)
        self.value = torch.zeros(n, device=dev)
        self.gmi = _one_instance()
        code = gmi.dtype_code("f32" if case["dtype"] == "f32" else "bf16")
        desc = gmi.model_desc(case["obs"], case["act"], _widths(case), code, n)
        if self.fp8:
            gmi.gmi_wait_stream(self.gmi)
            self.model = gmi.gmi_fp8_bind(self.gmi, desc)
            gmi.gmi_fp8_refresh(self.gmi, self.model, self.theta)
        else:
            size = gmi.gmi_model_shadow_bytes(desc)
            self.shadow = torch.zeros(size, dtype=torch.uint8, device=dev) if size else None
            gmi.gmi_wait_stream(self.gmi)
            self.model = gmi.gmi_model_bind(self.gmi, desc, self.theta, self.shadow)
            gmi.gmi_model_refresh_shadow(self.gmi, self.model)

    def step(self):
        call = gmi.agent_act_fp8 if self.fp8 else gmi.agent_act
        call(self.gmi, self.model, self.obs, self.n, self.seed, self.calls, 0, self.act, self.logp, self.value, self.mu)
        self.calls += 1
        return dict(act=self.act, logp=self.logp, value=self.value, mu=self.mu)

    def __del__(self):
        if hasattr(self, "model"):
            gmi.gmi_sync(self.gmi)
            (gmi.gmi_fp8_destroy if self.fp8 else gmi.gmi_model_destroy)(self.model)


class _Pipeline:
    def __init__(self, case, seed):
        rng = np.random.default_rng(seed)
        a_mat, b_mat = _env(case, rng)
        n = case["agents"]
        states = [rng.standard_normal((case["envs"], case["obs"]), dtype=np.float32) for _ in range(n)]
        probe = gmi.gmi_create()
        cus = gmi.gmi_cu_count(probe)
        gmi.gmi_destroy(probe)
        self.case, self.k = case, 0
        self.pipe = InstancePipeline(n_agents=n, n_envs=case["envs"], obs_dim=case["obs"], act_dim=case["act"],
                                     hidden=_widths(case), horizon=case["horizon"], dtype=case["dtype"],
                                     theta=_theta(case, rng), a_mat=a_mat, b_mat=b_mat, state0=states, noise_std=0.01,
                                     reward_scale=case["reward_scale"], done_period=0, done_threshold=(1 << 32) // 1000,
                                     seed=seed, minibatch=case["minibatch"],
                                     agent_masks=cu_masks(cus, [cus // n // 8 * 8] * n), host_ordered=True)
        self.states = [torch.tensor(s, device="cuda:0") for s in states]
        torch.cuda.synchronize()

    def step(self):
        p, c = self.pipe, self.case
        for ag, s in zip(p.agents, self.states):      # fresh environments, as above
            gmi.gmi_transfer(ag.gmi, ag.gmi, s, ag.obs[ag.cur], s.numel() * 4)
        p.iteration_sync(self.k, gamma=GAMMA, lam=LAM, epochs=c["epochs"], minibatch=c["minibatch"], **HYPER)
        self.k += 1
        b = p.bufs[0]
        return dict(theta=p.theta, adam_m=p.adam_m, adam_v=p.adam_v, obs=b.obs, act=b.act, logp=b.logp, val=b.val, rew=b.rew,
                    done=b.done, adv=b.adv, ret=b.ret, last_value=p.last_value[0])

    def __del__(self):
        if hasattr(self, "pipe"):
            self.pipe.close()


def prepare(case, seed):
    return {"train": _Train, "serve": _Serve, "pipeline": _Pipeline}[case["kind"]](case, seed)


def run(state):
    return state.step()


# ------------------------------------------------------------------------------------------------ measures
def work(case):
    """Products of the two networks (and of the environment's dynamics) at their own widths; every array that comes in
    read once and every array that goes out written once."""
    o, a = case["obs"], case["act"]
    mac = first = params = 0
    for out in (a, 1):
        prev = o
        for i, n in enumerate(_widths(case) + [out]):
            mac += prev * n
            first += prev * n if i == 0 else 0
            params += prev * n + n
            prev = n
    params += a
    if case["kind"] == "serve":
        n = case["rows"]
        weight = {"f32": 4, "bf16": 2, "fp8": 1}[case["dtype"]]
        return dict(bytes=weight * params + 4.0 * n * (o + 2 * a + 2), flops=2.0 * n * mac)
    envs = case["envs"] * case.get("agents", 1)
    samples = envs * case["horizon"]
    # collection: both nets per sample and the environment's product; update: forward, weight gradients, and input
    # gradients of every layer but the first
    flops = 2.0 * samples * (mac + o * (o + a)) + 2.0 * case["epochs"] * samples * (3 * mac - first)
    # environment states in and out, the experience with advantages and returns, parameters and both Adam moments
    data = 4.0 * envs * (2 * o + 3) + samples * (4.0 * (o + a + 5) + 1) + 24.0 * params
    return dict(bytes=data, flops=flops)


def tolerance(case):
    """fp32: order of 32-bit sums (after training also Adam's first steps, lr * sign(g), where a gradient is all
    rounding).  bf16: 8-bit mantissas of the operands.  fp8: an activation that rounds to the neighbouring 3-bit
    mantissa."""
    if case["kind"] == "serve":
        return {"f32": {"rel": 1e-5}, "bf16": {"rel": 1e-2}, "fp8": {"rel": 2e-2, "max": 0.3}}[case["dtype"]]
    return {"rel": 5e-5, "max": 1e-2} if case["dtype"] == "f32" else {"rel": 1e-2}
