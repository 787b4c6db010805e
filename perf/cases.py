"""The work that users of the learner-update library have it do, as cases to time and compare.

Kinds of case, each one call (or one learning phase) through the package's public entry points:

actor       impala_actor_step: what an actor does for every environment step (forward, Gumbel-max)
learner     learner_step: one whole learning phase, PPO (GAE, epochs x minibatches, Adam) or
            IMPALA (V-trace, env-block minibatches, RMSprop)
entry_fwd   a stage's entry, conv3x3 + max-pool (uint8 frames gathered by row index at stage 0)
block_fwd   a residual block's forward
block_bwd   a residual block's whole backward (input gradient and both weight gradients)
entry_bwd   a stage entry's whole backward from the pooled gradient
frames_bwd  the first stage entry's backward (weight gradient of the uint8 frames' conv)
conv_bwd    a 64-channel residual conv's whole backward (relu'd input, skip gradient added)

Everything is bf16 with float32 parameters, gradients and optimiser state, as the learner trains;
the library's float32 mode is a validation mode and no workload. The networks are the paper's
IMPALA-ResNet, (16, 32, 32) / 256, and its widened form, (32, 64, 64) / 512, on 84x84x4 frames;
drawn cases also take other frame sizes.
"""
from __future__ import annotations

from types import SimpleNamespace

import numpy as np
import torch
import torch.nn.functional as F

import paper_2310_00036_amd as P

DEV = "cuda:0"
BASE, WIDE = (16, 32, 32), (32, 64, 64)
GAMMA, LAM, CLIP, VF, ENT = 0.99, 0.95, 0.1, 0.5, 0.01


def listed():
    return [
        # eight evaluation environments stepped together: launches and latency
        dict(name="actor_b8", kind="actor", net="base", n=8, H=84, W=84, A=18),
        # one actor's environments, stepped together
        dict(name="actor_b128", kind="actor", net="base", n=128, H=84, W=84, A=18),
        # PPO, 64 environments x 128 steps, 4 minibatches of 2048 x 2 epochs: the benchmark's workload
        dict(name="ppo_64x128", kind="learner", algo="ppo", E=64, T=128, epochs=2, nmb=4, H=84, W=84, A=18),
        # the paper's IMPALA setting: 128 environments x 20 steps, 4 env-block minibatches, RMSprop
        dict(name="impala_128x20", kind="learner", algo="impala", E=128, T=20, epochs=1, nmb=4, H=84, W=84, A=18),
        # layers of one PPO minibatch (2048 frames) of the standard net
        dict(name="frames_entry_16", kind="entry_fwd", n=2048, H=84, W=84, ci=4, co=16),
        dict(name="block_fwd_16", kind="block_fwd", n=2048, H=42, W=42, ci=16, co=16),
        dict(name="block_fwd_32", kind="block_fwd", n=2048, H=21, W=21, ci=32, co=32),
        dict(name="block_bwd_16", kind="block_bwd", n=2048, H=42, W=42, ci=16, co=16),
        dict(name="entry_bwd_32", kind="entry_bwd", n=2048, H=42, W=42, ci=16, co=32),
        # layers of one IMPALA env block (32 environments x 20 steps: 640 frames)
        dict(name="block_bwd_32", kind="block_bwd", n=640, H=11, W=11, ci=32, co=32),
        dict(name="frames_bwd_16", kind="frames_bwd", n=640, H=84, W=84, ci=4, co=16),
        # the widened net's 8192-frame minibatch
        dict(name="wide_conv_bwd_64", kind="conv_bwd", n=8192, H=21, W=21, ci=64, co=64),
    ]


def draw(rng):
    """One more case: any kind, the networks' layers, frame counts over their whole range."""
    def log_int(lo, hi):
        return max(lo, min(hi, round(lo * (hi / lo) ** rng.random())))

    side = (84, 84) if rng.random() < 0.5 else (rng.randint(60, 96), rng.randint(60, 96))
    half = lambda hw, k: hw if k == 0 else half((-(-hw[0] // 2), -(-hw[1] // 2)), k - 1)  # noqa: E731
    kind = rng.choice(("actor", "learner", "entry_fwd", "block_fwd", "block_bwd", "entry_bwd", "frames_bwd", "conv_bwd"))
    if kind == "actor":
        return dict(kind=kind, net=rng.choice(("base", "wide")), n=log_int(1, 1024), H=side[0], W=side[1], A=rng.randint(4, 18))
    if kind == "learner":
        algo = rng.choice(("ppo", "impala"))
        nmb = rng.choice((1, 2, 4))
        E = nmb * log_int(2, 96 // nmb)
        T = rng.randint(8, 64) if algo == "ppo" else rng.randint(5, 40)
        return dict(kind=kind, algo=algo, E=E, T=T, epochs=rng.choice((1, 2)) if algo == "ppo" else 1, nmb=nmb,
                    H=side[0], W=side[1], A=rng.randint(4, 18))
    stage, ci, co = rng.choice({
        "entry_fwd": ((0, 4, 16), (0, 4, 32), (1, 16, 32), (2, 32, 32), (1, 32, 64), (2, 64, 64)),
        "block_fwd": ((1, 16, 16), (2, 32, 32), (3, 32, 32), (1, 32, 32)),
        "block_bwd": ((1, 16, 16), (2, 32, 32), (3, 32, 32), (1, 32, 32)),
        "entry_bwd": ((1, 16, 32), (2, 32, 32), (1, 32, 64), (2, 64, 64)),
        "frames_bwd": ((0, 4, 16), (0, 4, 32)),
        "conv_bwd": ((2, 64, 64), (3, 64, 64)),
    }[kind])
    H, W = half(side, stage)
    return dict(kind=kind, n=log_int(5, 8192), H=H, W=W, ci=ci, co=co)


# ------------------------------------------------------------------------------- inputs


def _gen(seed):
    return torch.Generator(device=DEV).manual_seed(int(seed))


def _net(case):
    ch, hidden = (WIDE, 512) if case.get("net") == "wide" else (BASE, 256)
    return SimpleNamespace(in_h=case["H"], in_w=case["W"], in_c=4, ch=ch, hidden=hidden, num_actions=case["A"])


def _params(net, g):
    """He-normal weights and zero biases; the policy head a hundredth and the value head a tenth
    as large, so that the policy still explores and the values have the size of returns."""
    parts = []
    for name, shape, _ in P.impala_param_layout(net):
        if name.endswith(".b"):
            parts.append(torch.zeros(int(np.prod(shape)), device=DEV))
            continue
        gain = {"logits.w": 0.01, "value.w": 0.1}.get(name, 1.0)
        w = torch.randn(int(np.prod(shape)), generator=g, device=DEV)
        parts.append(w * (gain * (2.0 / float(np.prod(shape[:-1]))) ** 0.5))
    return torch.cat(parts)


def _frames(g, n, H, W):
    return torch.randint(0, 256, (n, H, W, 4), dtype=torch.uint8, generator=g, device=DEV)


def _act(g, shape, scale=1.0):
    return (torch.randn(shape, generator=g, device=DEV) * scale).to(torch.bfloat16)


def _weights(g, ci, co):
    return torch.randn((3, 3, ci, co), generator=g, device=DEV) * (2.0 / (9 * ci)) ** 0.5


def _pool_arg(g, n, H, W, co):
    """The argmax (0..8, row-major in the window) of the max-pool over random conv outputs."""
    oh, ow = -(-H // 2), -(-W // 2)
    out = torch.empty((n, oh, ow, co), dtype=torch.uint8, device=DEV)
    for s in range(0, n, 256):
        c = torch.randn((min(256, n - s), H, W, co), generator=g, device=DEV)
        out[s:s + 256] = torch.stack(_windows(c, float("-inf"))).argmax(0).to(torch.uint8)
    return out


def _bytes(nbytes):
    return torch.empty(max(int(nbytes), 1), dtype=torch.uint8, device=DEV)


def _inputs(case, seed):
    """The tensors of a case, from the seed alone."""
    g = _gen(seed)
    kind, H, W = case["kind"], case["H"], case["W"]
    s = SimpleNamespace(case=case)
    if kind == "actor":
        s.net, n = _net(case), case["n"]
        s.params, s.obs = _params(s.net, g), _frames(g, n, H, W)
        s.gumbel = -torch.log(-torch.log(torch.rand((n, case["A"]), generator=g, device=DEV).clamp(1e-6, 1 - 1e-6)))
    elif kind == "learner":
        _rollout(s, case, g)
    else:
        n, ci, co = case["n"], case["ci"], case["co"]
        oh, ow = -(-H // 2), -(-W // 2)
        if kind in ("block_fwd", "block_bwd"):
            s.x, s.w1, s.w2 = _act(g, (n, H, W, ci)), _weights(g, ci, ci), _weights(g, ci, ci)
            s.b1, s.b2 = (torch.randn(ci, generator=g, device=DEV) * 0.1 for _ in range(2))
            if kind == "block_bwd":
                s.t, s.dy = _act(g, (n, H, W, ci)), _act(g, (n, H, W, ci), 1e-3)
        elif kind in ("entry_fwd", "frames_bwd"):
            # a minibatch's rows of a rollout four times as long (at least 64 frames)
            s.w, s.b = _weights(g, ci, co), torch.randn(co, generator=g, device=DEV) * 0.1
            if ci == 4:
                rows = max(64, min(4 * n, 8192))
                s.x = _frames(g, rows, H, W)
                s.rows = torch.randperm(rows, generator=g, device=DEV)[:n].to(torch.int32)
                if rows < n:
                    s.rows = torch.randint(0, rows, (n,), generator=g, device=DEV).to(torch.int32)
            else:
                s.x, s.rows = _act(g, (n, H, W, ci)), None
            if kind == "frames_bwd":
                s.dy, s.arg = _act(g, (n, oh, ow, co), 1e-3), _pool_arg(g, n, H, W, co)
        elif kind == "entry_bwd":
            s.x, s.w = _act(g, (n, H, W, ci)), _weights(g, ci, co)
            s.dy, s.arg = _act(g, (n, oh, ow, co), 1e-3), _pool_arg(g, n, H, W, co)
        else:
            s.x, s.w = _act(g, (n, H, W, ci)), _weights(g, ci, co)
            s.dy, s.add = _act(g, (n, H, W, co), 1e-3), _act(g, (n, H, W, ci), 1e-3)
    return s


def _rollout(s, case, g):
    """A rollout as an actor leaves it: uniform frames, clipped rewards, actions sampled from the
    initial policy with their log-probs (PPO: and values), the behaviour policy a little off."""
    net = s.net = _net(case)
    T, E, A, ppo = case["T"], case["E"], case["A"], case["algo"] == "ppo"
    n = T * E
    s.params = _params(net, g)
    s.obs = _frames(g, n + E, case["H"], case["W"])
    with torch.no_grad():
        z, v = _apply(net, s.params, s.obs, torch.float32)
    if not ppo:
        z = z + 0.3 * torch.randn(z.shape, generator=g, device=DEV)
    s.actions = torch.multinomial(torch.softmax(z[:n], 1), 1, generator=g)[:, 0].to(torch.int32)
    s.logp = torch.log_softmax(z[:n], 1).gather(1, s.actions.long()[:, None])[:, 0].contiguous()
    s.values, s.next_value = (v[:n].contiguous(), v[n:].contiguous()) if ppo else (None, None)
    u = torch.rand((T, E), generator=g, device=DEV)
    s.rewards = (u > 0.95).float() - (u < 0.05).float()
    s.dones = (torch.rand((T, E), generator=g, device=DEV) < 0.02).to(torch.uint8)
    s.next_done = (torch.rand(E, generator=g, device=DEV) < 0.02).to(torch.uint8)
    s.perm = None
    if ppo:
        s.obs = s.obs[:n].contiguous()
        s.perm = torch.stack([torch.randperm(n, generator=g, device=DEV) for _ in range(case["epochs"])]).to(torch.int32)
    wl = SimpleNamespace(algo=case["algo"], T=T, E=E, epochs=case["epochs"], num_minibatches=case["nmb"],
                         mb=n // case["nmb"], norm_adv=1, gamma=GAMMA, lam=LAM if ppo else 1.0, clip_eps=CLIP,
                         vf_coef=VF, ent_coef=ENT, pg_coef=1.0, rho_bar=1.0, c_bar=1.0, pg_rho_bar=1.0,
                         lr=2.5e-4 if ppo else 6e-4, beta1=0.9, beta2=0.999, adam_eps=1e-5,
                         max_grad_norm=0.5 if ppo else 40.0, optimizer="adam" if ppo else "rmsprop",
                         rms_decay=0.99, rms_eps=0.01)
    s.wl, s.updates = wl, case["epochs"] * case["nmb"]


def prepare(case, seed):
    s = _inputs(case, seed)
    kind, H, W, prec = case["kind"], case["H"], case["W"], P.PREC_BF16
    f32 = lambda *shape: torch.empty(shape, device=DEV)  # noqa: E731
    b16 = lambda *shape: torch.empty(shape, dtype=torch.bfloat16, device=DEV)  # noqa: E731
    if kind == "actor":
        n = case["n"]
        s.ws = _bytes(P.impala_workspace_bytes(s.net, n, prec, 0))
        s.actions = torch.empty(n, dtype=torch.int32, device=DEV)
        s.logp, s.value, s.logits = f32(n), f32(n), f32(n, case["A"])
        return s
    if kind == "learner":
        s.cfg = P.learner_cfg(s.wl, prec)
        s.ws = _bytes(P.learner_workspace_bytes(s.net, s.cfg))
        s.m, s.v, s.step = torch.zeros_like(s.params), torch.zeros_like(s.params), 0
        s.stats = f32(s.updates, 8)
        s.rollout = P.rollout_struct(s.obs, s.actions, s.logp, s.rewards, s.dones, s.values, s.next_value, s.next_done)
        return s
    n, ci, co = case["n"], case["ci"], case["co"]
    oh, ow = -(-H // 2), -(-W // 2)
    if kind == "block_fwd":
        s.t, s.y = b16(n, H, W, ci), b16(n, H, W, ci)
    elif kind == "entry_fwd":
        s.y, s.arg = b16(n, oh, ow, co), torch.empty((n, oh, ow, co), dtype=torch.uint8, device=DEV)
    else:
        s.dx = b16(n, H, W, ci)
        s.dw, s.db = f32(3, 3, ci, co), f32(co)
        if kind == "block_bwd":
            s.dw2, s.db2 = f32(3, 3, ci, co), f32(co)
            s.ws = _bytes(P.impala_resblock_bwd_workspace_bytes(prec, ci))
        elif kind == "frames_bwd":
            s.ws = _bytes(P.impala_conv3x3_pool_wgrad_u8_workspace_bytes(prec, co))
        else:
            s.ws = _bytes(P.impala_conv3x3_bwd_workspace_bytes(prec, ci, co))
    return s


def run(s):
    case, prec = s.case, P.PREC_BF16
    kind, H, W = case["kind"], case["H"], case["W"]
    if kind == "actor":
        P.impala_actor_step(s.net, prec, s.params, s.obs, case["n"], s.gumbel, s.ws, s.actions, s.logp, s.value, s.logits)
        return dict(actions=s.actions, logp=s.logp, value=s.value, logits=s.logits)
    if kind == "learner":
        # the optimiser's moments are left out of what is compared: they are the raw bf16 gradient,
        # which a change of rounding anywhere in the forward pass turns by several percent (pool and
        # ReLU decisions); the updated weights carry the same update
        s.step = P.learner_step(s.net, s.cfg, s.rollout, s.params, s.m, s.v, s.step, s.perm, s.ws, s.stats)
        return dict(params=s.params, stats=s.stats)
    n, ci, co = case["n"], case["ci"], case["co"]
    if kind == "block_fwd":
        P.impala_resblock_fwd(prec, n, H, W, ci, s.x, s.w1, s.b1, s.w2, s.b2, s.t, s.y)
        return dict(t=s.t, y=s.y)
    if kind == "block_bwd":
        P.impala_resblock_bwd(prec, n, H, W, ci, s.dy, s.t, s.x, s.w1, s.w2, s.dx, s.dw, s.db, s.dw2, s.db2, s.ws)
        return dict(dx=s.dx, dwa=s.dw, dba=s.db, dwb=s.dw2, dbb=s.db2)
    if kind == "entry_fwd":
        P.impala_conv3x3_pool_fwd(prec, n, H, W, ci, co, s.x, P.X_U8 if ci == 4 else P.X_PLAIN, s.rows, s.w, s.b, s.y, s.arg)
        return dict(y=s.y, arg=s.arg)
    if kind == "frames_bwd":
        P.impala_conv3x3_pool_wgrad_u8(prec, n, H, W, co, s.x, s.rows, s.dy, s.arg, s.dw, s.db, s.ws)
        return dict(dw=s.dw, db=s.db)
    if kind == "entry_bwd":
        P.impala_conv3x3_bwd(prec, n, H, W, ci, co, s.dy, s.x, P.X_PLAIN, s.w, None, s.dx, s.dw, s.db, s.ws, pool_arg=s.arg)
    else:
        P.impala_conv3x3_bwd(prec, n, H, W, ci, co, s.dy, s.x, P.X_RELU, s.w, s.add, s.dx, s.dw, s.db, s.ws)
    return dict(dx=s.dx, dw=s.dw, db=s.db)


# ------------------------------------------------------------------------------- work


def _net_macs(net):
    """(multiply-adds of one frame's forward, of its first conv)."""
    h, w, ci, macs, first = net.in_h, net.in_w, 4, 0, 0
    for c in net.ch:
        macs += h * w * 9 * ci * c
        first = first or macs
        h, w, ci = -(-h // 2), -(-w // 2), c
        macs += 4 * h * w * 9 * c * c
    return macs + h * w * ci * net.hidden + net.hidden * (net.num_actions + 1), first


def work(case):
    kind, H, W = case["kind"], case["H"], case["W"]
    if kind in ("actor", "learner"):
        net = _net(case)
        macs, first = _net_macs(net)
        params = P.impala_param_count(net)
        if kind == "actor":
            n = case["n"]
            return dict(bytes=n * (H * W * 4 + 8 * case["A"] + 12) + 4 * params, flops=2 * n * macs)
        n, passes = case["T"] * case["E"], case["epochs"]
        boot = case["E"] if case["algo"] == "impala" else 0
        # each pass reads the frames once; the rollout arrays once; the optimiser's state both ways
        state = 12 if case["algo"] == "ppo" else 8
        return dict(bytes=(passes * n + boot) * H * W * 4 + 25 * n + 2 * state * params,
                    flops=passes * n * 2 * (3 * macs - first) + boot * 2 * macs)
    n, ci, co = case["n"], case["ci"], case["co"]
    px, pooled = n * H * W, n * -(-H // 2) * -(-W // 2)
    conv = 2 * px * 9 * ci * co
    wb = 4 * 9 * ci * co
    if kind == "block_fwd":
        return dict(bytes=px * ci * 2 * 3 + 2 * wb, flops=2 * conv)
    if kind == "block_bwd":
        return dict(bytes=px * ci * 2 * 4 + 4 * wb, flops=4 * conv)
    if kind == "entry_fwd":
        return dict(bytes=px * ci * (1 if ci == 4 else 2) + pooled * co * 3 + wb, flops=conv)
    if kind == "frames_bwd":
        return dict(bytes=px * ci + pooled * co * 3 + wb, flops=conv)
    if kind == "entry_bwd":
        return dict(bytes=px * ci * 2 * 2 + pooled * co * 3 + 2 * wb, flops=2 * conv)
    return dict(bytes=px * 2 * (3 * ci + co) + 2 * wb, flops=2 * conv)


def tolerance(case):
    """Largest relative error of another correct bf16 implementation: four times what a layer's
    outputs were measured off the 64-bit result (forward and input gradients 2.0e-3 .. 2.7e-3,
    the frames' weight gradient 1.3e-3). Whole calls: values 2e-2 .. 3e-2 (sums that cancel),
    logits 6e-3, the updates' statistics 2e-3 .. 5e-2, new weights 3e-4; whole numbers that
    rounding may turn: sampled actions, pool argmaxes."""
    return {
        "actor": {"rel": 0.03, "differ": 0.01},
        "learner": {"rel": 0.03},
        "entry_fwd": {"rel": 0.01, "differ": 0.01},
        "frames_bwd": {"rel": 0.005},
    }.get(case["kind"], {"rel": 0.01})


# ------------------------------------------------------------------------------- 64-bit results


def _windows(x, fill):
    """The nine stride-2 views of a SAME 3x3 max-pool over [n, H, W, C] (padding split low = P // 2)."""
    H, W = x.shape[1:3]
    oh, ow = -(-H // 2), -(-W // 2)
    ph, pw = (oh - 1) * 2 + 3 - H, (ow - 1) * 2 + 3 - W
    xp = F.pad(x, (0, 0, pw // 2, pw - pw // 2, ph // 2, ph - ph // 2), value=fill)
    return [xp[:, i:i + 2 * oh - 1:2, j:j + 2 * ow - 1:2] for i in range(3) for j in range(3)]


def _pool(x):
    y, arg = torch.stack(_windows(x, float("-inf"))).max(0)
    return y, arg


def _unpool(dy, arg, H, W):
    """The max-pool's input gradient."""
    n, C = dy.shape[0], dy.shape[3]
    oh, ow = dy.shape[1:3]
    ph, pw = (oh - 1) * 2 + 3 - H, (ow - 1) * 2 + 3 - W
    dxp = dy.new_zeros((n, H + ph, W + pw, C))
    for k in range(9):
        i, j = divmod(k, 3)
        dxp[:, i:i + 2 * oh - 1:2, j:j + 2 * ow - 1:2] += torch.where(arg == k, dy, 0)
    return dxp[:, ph // 2:ph // 2 + H, pw // 2:pw // 2 + W]


def _cols(x):
    """[n, H, W, C] -> [n*H*W, 9*C]: the zero-padded 3x3 neighbourhoods, tap-major."""
    n, H, W, C = x.shape
    xp = F.pad(x, (0, 0, 1, 1, 1, 1))
    return torch.cat([xp[:, i:i + H, j:j + W] for i in range(3) for j in range(3)], 3).reshape(n * H * W, 9 * C)


def _conv(x, w, b=None):
    n, H, W, _ = x.shape
    y = (_cols(x) @ w.reshape(-1, w.shape[3])).reshape(n, H, W, w.shape[3])
    return y if b is None else y + b


def _conv_t(dy, w):
    return _conv(dy, w.flip(0, 1).transpose(2, 3))


def _wgrad(x, dy):
    co = dy.shape[3]
    return (_cols(x).t() @ dy.reshape(-1, co)).reshape(3, 3, x.shape[3], co), dy.sum((0, 1, 2))


def _apply(net, params, obs, dtype, chunk=256):
    """Logits and values of frames; differentiable in params where they need a gradient."""
    W = {name: params[off:off + int(np.prod(shape))].reshape(shape).to(dtype)
         for name, shape, off in P.impala_param_layout(net)}
    zs, vs = [], []
    for s in range(0, obs.shape[0], chunk):
        x = obs[s:s + chunk].to(dtype) / 255
        for st in range(3):
            x, _ = _pool(_conv(x, W[f"s{st}.conv.w"], W[f"s{st}.conv.b"]))
            for r in range(2):
                t = _conv(x.relu(), W[f"s{st}.res{r}.conv0.w"], W[f"s{st}.res{r}.conv0.b"])
                x = x + _conv(t.relu(), W[f"s{st}.res{r}.conv1.w"], W[f"s{st}.res{r}.conv1.b"])
        h = (x.relu().reshape(x.shape[0], -1) @ W["dense.w"] + W["dense.b"]).relu()
        zs.append(h @ W["logits.w"] + W["logits.b"])
        vs.append((h @ W["value.w"])[:, 0] + W["value.b"])
    return torch.cat(zs), torch.cat(vs)


def _by_frames(n, px, f):
    """f(a, b) over chunks of frames; per-frame outputs joined, sums added (f: (joined, summed))."""
    step = max(1, int(4e8 / px))
    joined, summed = None, None
    for a in range(0, n, step):
        j, q = f(a, min(n, a + step))
        joined = [[x] for x in j] if joined is None else [u + [x] for u, x in zip(joined, j)]
        summed = q if summed is None else [u + x for u, x in zip(summed, q)]
    return [torch.cat(u) for u in joined], summed


def _exact_learner(s):
    """learner_step in 64 bits: the new parameters and the updates' statistics."""
    net, wl, T, E = s.net, s.wl, s.wl.T, s.wl.E
    n, dt = T * E, torch.float64
    p, m, v = s.params.to(dt), torch.zeros_like(s.params, dtype=dt), torch.zeros_like(s.params, dtype=dt)
    live = 1 - torch.cat([s.dones[1:], s.next_done[None]]).to(dt)
    rew, acts, behav = s.rewards.to(dt), s.actions.long(), s.logp.to(dt)
    if wl.algo == "ppo":
        val = s.values.to(dt).reshape(T, E)
        nxt = torch.cat([val[1:], s.next_value.to(dt)[None]])
        adv, run_ = torch.zeros_like(val), torch.zeros(E, dtype=dt, device=DEV)
        for t in reversed(range(T)):
            run_ = rew[t] + wl.gamma * live[t] * nxt[t] - val[t] + wl.gamma * wl.lam * live[t] * run_
            adv[t] = run_
        adv, ret = adv.reshape(-1), (adv + val).reshape(-1)
    out = []
    for u in range(s.updates):
        if wl.algo == "ppo":
            rows = s.perm[u // wl.num_minibatches, u % wl.num_minibatches * wl.mb:][:wl.mb].long()
        else:
            eb = E // wl.num_minibatches
            envs = torch.arange(u * eb, (u + 1) * eb, device=DEV)
            rows = (torch.arange(T + 1, device=DEV)[:, None] * E + envs).reshape(-1)
        k = rows.numel() if wl.algo == "ppo" else T * eb
        with torch.no_grad():
            z, val = _apply(net, p, s.obs[rows], dt)
        z.requires_grad_(True)
        val.requires_grad_(True)
        lp = torch.log_softmax(z[:k], 1)
        a_lp = lp.gather(1, acts[rows[:k], None])[:, 0]
        ent = -(lp.exp() * lp).sum(1).mean()
        if wl.algo == "ppo":
            a, tgt = adv[rows], ret[rows]
            ah = (a - a.mean()) / (a.std(unbiased=False) + 1e-8)
            ratio = (a_lp - behav[rows]).exp()
            pg = torch.maximum(-ah * ratio, -ah * ratio.clamp(1 - wl.clip_eps, 1 + wl.clip_eps)).mean()
            extra = [((ratio - 1) - ratio.log()).mean(), ((ratio - 1).abs() > wl.clip_eps).to(dt).mean()]
        else:
            with torch.no_grad():
                V = val.reshape(T + 1, eb)
                rho = (a_lp - behav[rows[:k]]).exp().reshape(T, eb).clamp(max=1.0)
                disc, r = wl.gamma * live[:, envs], rew[:, envs]
                vs, q = V.clone(), torch.zeros_like(rho)
                for t in reversed(range(T)):
                    vs[t] = V[t] + rho[t] * (r[t] + disc[t] * V[t + 1] - V[t]) + disc[t] * rho[t] * (vs[t + 1] - V[t + 1])
                    q[t] = rho[t] * (r[t] + disc[t] * vs[t + 1] - V[t])
                tgt, q = vs[:T].reshape(-1), q.reshape(-1)
            pg = (-q * a_lp).mean()
            extra = [q.mean(), tgt.mean()]
        vl = 0.5 * (val[:k] - tgt).square().mean()
        loss = pg + wl.vf_coef * vl - wl.ent_coef * ent
        dz, dv = torch.autograd.grad(loss, (z, val))
        grad = torch.zeros_like(p)
        for c in range(0, k, 256):
            q_ = p.clone().requires_grad_(True)
            zc, vc = _apply(net, q_, s.obs[rows[c:min(k, c + 256)]], dt)
            grad += torch.autograd.grad((zc, vc), q_, (dz[c:c + len(zc)], dv[c:c + len(zc)]))[0]
        norm = grad.norm()
        out.append(torch.stack([loss, pg, vl, ent, *extra, norm, torch.zeros_like(norm)]).detach())
        g = grad * (wl.max_grad_norm / norm).clamp(max=1.0)
        if wl.optimizer == "adam":
            m, v = wl.beta1 * m + (1 - wl.beta1) * g, wl.beta2 * v + (1 - wl.beta2) * g * g
            p = p - wl.lr * (m / (1 - wl.beta1 ** (u + 1))) / ((v / (1 - wl.beta2 ** (u + 1))).sqrt() + wl.adam_eps)
        else:
            v = wl.rms_decay * v + (1 - wl.rms_decay) * g * g
            p = p - wl.lr * g / (v + wl.rms_eps).sqrt()
    return dict(params=p, stats=torch.stack(out))


def exact(case, seed):
    s = _inputs(case, seed)
    kind, dt = case["kind"], torch.float64
    if kind == "actor":
        with torch.no_grad():
            z, v = _apply(s.net, s.params, s.obs, dt)
        a = (z + s.gumbel).argmax(1)
        return dict(actions=None, logp=torch.log_softmax(z, 1).gather(1, a[:, None])[:, 0], value=v, logits=z)
    if kind == "learner":
        return _exact_learner(s)
    n, H, W, ci, co = case["n"], case["H"], case["W"], case["ci"], case["co"]
    px = H * W * 9 * max(ci, co)
    if kind == "block_fwd":
        def f(a, b):
            x = s.x[a:b].to(dt)
            t = _conv(x.relu(), s.w1.to(dt), s.b1)
            return (t, x + _conv(t.relu(), s.w2.to(dt), s.b2)), []
        (t, y), _ = _by_frames(n, px, f)
        return dict(t=t, y=y)
    if kind == "block_bwd":
        def f(a, b):
            x, t, dy = s.x[a:b].to(dt), s.t[a:b].to(dt), s.dy[a:b].to(dt)
            dt_ = _conv_t(dy, s.w2.to(dt)) * (t > 0)
            dx = _conv_t(dt_, s.w1.to(dt)) * (x > 0) + dy
            return (dx,), [*_wgrad(x.relu(), dt_), *_wgrad(t.relu(), dy)]
        (dx,), q = _by_frames(n, px, f)
        return dict(dx=dx, dwa=q[0], dba=q[1], dwb=q[2], dbb=q[3])
    frame = (lambda a, b: s.x[s.rows[a:b].long()].to(dt) / 255) if ci == 4 else (lambda a, b: s.x[a:b].to(dt))
    if kind == "entry_fwd":
        (y,), _ = _by_frames(n, px, lambda a, b: ((_pool(_conv(frame(a, b), s.w.to(dt), s.b))[0],), []))
        return dict(y=y, arg=None)

    def f(a, b):
        x, dy = frame(a, b), s.dy[a:b].to(dt)
        if kind == "conv_bwd":
            return ((_conv_t(dy, s.w.to(dt)) * (x > 0) + s.add[a:b].to(dt)),), list(_wgrad(x.relu(), dy))
        dc = _unpool(dy, s.arg[a:b], H, W)
        dx = _conv_t(dc, s.w.to(dt)) if kind == "entry_bwd" else dy.new_zeros(1)
        return (dx,), list(_wgrad(x, dc))
    (dx,), (dw, db) = _by_frames(n, px, f)
    return dict(dw=dw, db=db) if kind == "frames_bwd" else dict(dx=dx, dw=dw, db=db)
