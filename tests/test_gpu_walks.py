"""The column-walk kernels against the per-layer calls they stand for, at the edges of their tile
shapes: rows and columns around a walk's group of 16 anchors, whole frames and bands, a ragged last
tile, row pitches of both parities, windows near the LDS budget, and pointers that are aligned to
four bytes only. A walk adds the products of one output in the per-layer kernels' order, so stored
outputs are equal bit for bit; weight gradients are float32 sums in another order."""
from __future__ import annotations

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

SHAPES = [(1, 1, 1), (2, 2, 5), (7, 3, 3), (33, 4, 7), (5, 11, 11), (17, 11, 11), (700, 11, 11), (33, 21, 21),
          (3, 21, 22), (9, 8, 15), (2, 42, 42), (515, 42, 42), (1, 43, 39), (600, 5, 7), (3, 64, 64), (1, 7, 97),
          # the networks' layers at an actor's and an IMPALA block's frames
          (128, 21, 21), (150, 42, 42), (640, 21, 21), (640, 11, 11), (2048, 11, 11),
          # the row counts per walk (each a kernel of its own) that those above leave out
          (65, 19, 26), (111, 17, 22), (550, 7, 15), (57, 9, 27), (85, 12, 22), (212, 7, 22), (37, 9, 31), (134, 17, 34),
          (77, 13, 30), (61, 4, 9), (48, 7, 22)]

# 64 channels, too wide for the walk's windows: the conv backward with specialised waves
WIDE64 = [(2, 5, 106), (1, 4, 107), (3, 9, 107)]
# 16 channels, taken tile by tile: whole bands and a ragged last one, whole frames, odd widths
TILES16 = [(515, 9, 97), (900, 11, 82), (200, 43, 103), (900, 29, 34), (4096, 9, 49), (4096, 21, 22), (3001, 38, 33)]

# the 32-channel forward: the widest that a walk's windows take, and wider
WIDE32 = [(2, 9, 139), (1, 1, 200), (1200, 7, 150), (3, 2, 140), (2, 5, 151), (3, 3, 256), (2, 1, 256), (300, 6, 141)]


def _p():
    import paper_2310_00036_amd as P
    return P


def _act(g, shape, offset=0):
    """bf16 normals; with `offset`, a view that many elements into its storage."""
    n = int(np.prod(shape))
    x = torch.randn(n + offset, generator=g, device="cuda:0").to(torch.bfloat16)
    return x[offset:].view(shape)


def _bits(x):
    return x.view(torch.int16)


@pytest.mark.parametrize("case", SHAPES + WIDE32, ids=lambda c: "n%d_%dx%d" % c)
@pytest.mark.parametrize("offset", [0, 2])
def test_resblock32_forward_equals_two_convolutions(case, offset):
    P = _p()
    n, H, W = case
    g = torch.Generator(device="cuda:0").manual_seed(n * 1009 + H * 31 + W)
    x = _act(g, (n, H, W, 32), offset)
    wpad = offset // 2   # weights one float off 16-byte alignment
    w1, w2 = ((torch.randn(9 * 32 * 32 + wpad, generator=g, device="cuda:0") * 0.1)[wpad:].view(3, 3, 32, 32)
              for _ in range(2))
    b1, b2 = (torch.randn(32, generator=g, device="cuda:0") for _ in range(2))
    b2 = None if offset else b2
    t, y, t_ref, y_ref = (torch.full((n * H * W * 32 + offset,), 7.0, device="cuda:0").to(torch.bfloat16)[offset:]
                          .view(n, H, W, 32) for _ in range(4))
    P.impala_resblock_fwd(P.PREC_BF16, n, H, W, 32, x, w1, b1, w2, b2, t, y)
    P.impala_conv3x3_fwd(P.PREC_BF16, n, H, W, 32, 32, x, P.X_RELU, None, w1, b1, None, t_ref)
    P.impala_conv3x3_fwd(P.PREC_BF16, n, H, W, 32, 32, t_ref, P.X_RELU, None, w2, b2, x, y_ref)
    torch.cuda.synchronize()
    assert torch.equal(_bits(t), _bits(t_ref))
    assert torch.equal(_bits(y), _bits(y_ref))


@pytest.mark.parametrize("offset", [0, 2])
@pytest.mark.parametrize("C,case", [(C, c) for C in (16, 32) for c in SHAPES] + [(16, c) for c in TILES16],
                         ids=lambda c: "n%d_%dx%d" % c if isinstance(c, tuple) else "c%d" % c)
def test_resblock_backward_equals_two_conv_backwards(case, offset, C):
    P = _p()
    n, H, W = case
    g = torch.Generator(device="cuda:0").manual_seed(n * 1013 + H * 37 + W)
    dy, t, x = (_act(g, (n, H, W, C), offset) for _ in range(3))
    wpad = offset // 2
    wa, wb = ((torch.randn(9 * C * C + wpad, generator=g, device="cuda:0") * 0.1)[wpad:].view(3, 3, C, C)
              for _ in range(2))
    dx, dt, dx_ref = (torch.full((n * H * W * C + offset,), 7.0, device="cuda:0").to(torch.bfloat16)[offset:]
                      .view(n, H, W, C) for _ in range(3))
    gw = [torch.full(s, 9.0, device="cuda:0") for s in ((3, 3, C, C), (C,)) * 4]
    ws = torch.empty(max(P.impala_resblock_bwd_workspace_bytes(0, C), P.impala_conv3x3_bwd_workspace_bytes(0, C, C)),
                     dtype=torch.uint8, device="cuda:0")
    P.impala_resblock_bwd(P.PREC_BF16, n, H, W, C, dy, t, x, wa, wb, dx, *gw[:4], ws)
    P.impala_conv3x3_bwd(P.PREC_BF16, n, H, W, C, C, dy, t, P.X_RELU, wb, None, dt, gw[6], gw[7], ws)
    P.impala_conv3x3_bwd(P.PREC_BF16, n, H, W, C, C, dt, x, P.X_RELU, wa, dy, dx_ref, gw[4], gw[5], ws)
    torch.cuda.synchronize()
    assert torch.equal(_bits(dx), _bits(dx_ref))
    for got, want in zip(gw[:4], gw[4:]):
        # float32 sums of the same products in another order: the error of each is below 2^-20 of
        # the sum of their magnitudes, which for these normals is about sqrt(terms) times the sum
        scale = float(n * H * W) ** 0.5 * 0.5 + 1.0
        assert torch.allclose(got, want, rtol=1e-5, atol=2.0 ** -20 * scale * max(float(n * H * W) ** 0.5, 1.0))


@pytest.mark.parametrize("C,case", [(16, (33, 21, 21)), (16, (5, 42, 42)), (16, (900, 29, 34)), (32, (17, 11, 11)), (32, (3, 21, 22))],
                         ids=lambda c: "n%d_%dx%d" % c if isinstance(c, tuple) else "c%d" % c)
def test_resblock_backward_of_infinities(case, C):
    """dx equals two conv backwards' also where dy, t or x hold infinities and NaNs: neither padding nor the
    k-values past the ninth tap (zero weights) may turn an infinite value into a NaN."""
    P = _p()
    n, H, W = case
    g = torch.Generator(device="cuda:0").manual_seed(n * 7 + H * 3 + W)
    dy, t, x = (_act(g, (n, H, W, C)) for _ in range(3))
    bad = torch.tensor([float("inf"), -float("inf"), float("nan")], device="cuda:0").to(torch.bfloat16)
    for q in (dy, t, x):
        k = max(3, q.numel() // 20000)
        at = torch.randint(0, q.numel(), (k,), generator=g, device="cuda:0")
        q.view(-1)[at] = bad[torch.arange(k, device="cuda:0") % 3]
        q[0, 0, 0, 0], q[-1, -1, -1, -1] = bad[0], bad[1]   # the first and the last pixel
    wa, wb = (torch.randn((3, 3, C, C), generator=g, device="cuda:0") * 0.1 for _ in range(2))
    dx, dt, dx_ref = (torch.empty_like(x) for _ in range(3))
    gw = [torch.empty(s, device="cuda:0") for s in ((3, 3, C, C), (C,)) * 2]
    ws = torch.empty(max(P.impala_resblock_bwd_workspace_bytes(0, C), P.impala_conv3x3_bwd_workspace_bytes(0, C, C)),
                     dtype=torch.uint8, device="cuda:0")
    P.impala_resblock_bwd(P.PREC_BF16, n, H, W, C, dy, t, x, wa, wb, dx, *gw, ws)
    P.impala_conv3x3_bwd(P.PREC_BF16, n, H, W, C, C, dy, t, P.X_RELU, wb, None, dt, gw[0], gw[1], ws)
    P.impala_conv3x3_bwd(P.PREC_BF16, n, H, W, C, C, dt, x, P.X_RELU, wa, dy, dx_ref, gw[0], gw[1], ws)
    torch.cuda.synchronize()
    nan = torch.isnan(dx_ref)
    assert torch.isinf(dx_ref).any() and not nan.all()
    assert torch.equal(torch.isnan(dx), nan)
    assert torch.equal(_bits(dx)[~nan], _bits(dx_ref)[~nan])


@pytest.mark.parametrize("n", [1, 7, 8, 63, 64, 65])
def test_dense_layer_on_few_frames(n):
    """The dense GEMM at and around the frame count where its tiles are mostly empty: the
    forward's logits and values against those of the same frames in a batch of 128."""
    from synth import NetShape, draw_params
    P = _p()
    net = NetShape(num_actions=6)
    params = torch.from_numpy(draw_params(net, 11)).cuda()
    g = torch.Generator(device="cuda:0").manual_seed(n)
    obs = torch.randint(0, 256, (n, 84, 84, 4), dtype=torch.uint8, generator=g, device="cuda:0")
    big = torch.cat([obs, obs[:1].expand(128 - n, -1, -1, -1)]).contiguous()   # the same frames among 128
    out = []
    for k, o in ((n, obs), (128, big)):
        ws = torch.empty(P.impala_workspace_bytes(net, k, P.PREC_BF16, 0), dtype=torch.uint8, device="cuda:0")
        z, v = torch.empty((k, 6), device="cuda:0"), torch.empty(k, device="cuda:0")
        P.impala_cnn_fwd(net, P.PREC_BF16, params, o, None, k, ws, 0, z, v)
        out.append(torch.cat([z[:n], v[:n, None]], 1).double())
    torch.cuda.synchronize()
    # h is bf16: its rounding may turn where the k-splits' float32 sums differ, by one part in 2^8 of
    # single hidden units
    err = (out[0] - out[1]).norm() / out[1].norm()
    assert err <= 2.0 ** -8, err


@pytest.mark.parametrize("n", [1, 8, 63])
@pytest.mark.parametrize("hidden", [1024, 2056])
def test_dense_input_gradient_on_few_frames(n, hidden):
    """A hidden layer of 1024 units or more: the dense layer's input gradient on fewer than 64 frames, against
    the same frames among 128 whose other frames have no gradient."""
    from types import SimpleNamespace
    P = _p()
    net = SimpleNamespace(in_h=32, in_w=36, in_c=4, ch=(16, 32, 32), hidden=hidden, num_actions=6)
    g = torch.Generator(device="cuda:0").manual_seed(n + hidden)
    params = torch.randn(P.impala_param_count(net), generator=g, device="cuda:0") * 0.05
    obs = torch.randint(0, 256, (128, 32, 36, 4), generator=g, device="cuda:0", dtype=torch.int32).to(torch.uint8)
    dz, dv = torch.randn((128, 6), generator=g, device="cuda:0"), torch.randn(128, generator=g, device="cuda:0")
    dz[n:], dv[n:] = 0, 0
    ws, grads = {}, {}
    for k in (128, n):
        ws[k] = torch.empty(P.impala_workspace_bytes(net, k, P.PREC_BF16, 1), dtype=torch.uint8, device="cuda:0")
        z, v = torch.empty((k, 6), device="cuda:0"), torch.empty(k, device="cuda:0")
        P.impala_cnn_fwd(net, P.PREC_BF16, params, obs, None, k, ws[k], 1, z, v)
        grads[k] = torch.empty_like(params)
    # one forward's activations serve both (a forward on n frames rounds h its own way)
    for (name, off, _, _, _), (_, o, size, _, shape) in zip(P.impala_activation_layout(net, P.PREC_BF16, 128),
                                                            P.impala_activation_layout(net, P.PREC_BF16, n)):
        assert shape[0] == n, name
        ws[n][o:o + size] = ws[128][off:off + size]
    for k in (128, n):
        P.impala_cnn_bwd(net, P.PREC_BF16, params, obs, None, k, ws[k], dz, dv, grads[k])
    torch.cuda.synchronize()
    # dx is bf16: its rounding turns where the float32 sums of another split differ, and travels through the
    # trunk's bf16 gradients: each tensor within one part in 2^8
    for name, shape, off in P.impala_param_layout(net):
        a, b = (grads[k][off:off + int(np.prod(shape))].double() for k in (128, n))
        assert (a - b).norm() <= 2.0 ** -8 * a.norm() + 1e-30, name


@pytest.mark.parametrize("case", SHAPES + WIDE64, ids=lambda c: "n%d_%dx%d" % c)
@pytest.mark.parametrize("add", [False, True])
def test_conv64_backward_equals_input_and_weight_gradient(case, add):
    P = _p()
    n, H, W = case
    off = 2 if add else 0
    g = torch.Generator(device="cuda:0").manual_seed(n * 1019 + H * 41 + W)
    dy, x, skip = (_act(g, (n, H, W, 64), off) for _ in range(3))
    skip = skip if add else None
    w = (torch.randn(9 * 64 * 64 + off // 2, generator=g, device="cuda:0") * 0.1)[off // 2:].view(3, 3, 64, 64)
    dx, dx_ref = (torch.full((n * H * W * 64 + off,), 7.0, device="cuda:0").to(torch.bfloat16)[off:]
                  .view(n, H, W, 64) for _ in range(2))
    gw = [torch.full(s, 9.0, device="cuda:0") for s in ((3, 3, 64, 64), (64,)) * 2]
    ws = torch.empty(max(P.impala_conv3x3_bwd_workspace_bytes(0, 64, 64),
                         P.impala_conv3x3_wgrad_workspace_bytes(0, H, W, 64, 64)), dtype=torch.uint8, device="cuda:0")
    P.impala_conv3x3_bwd(P.PREC_BF16, n, H, W, 64, 64, dy, x, P.X_RELU, w, skip, dx, gw[0], gw[1], ws)
    P.impala_conv3x3_dgrad(P.PREC_BF16, n, H, W, 64, 64, dy, w, x, skip, dx_ref)
    P.impala_conv3x3_wgrad(P.PREC_BF16, n, H, W, 64, 64, x, P.X_RELU, None, dy, gw[2], gw[3], ws)
    torch.cuda.synchronize()
    assert torch.equal(_bits(dx), _bits(dx_ref))
    for got, want in zip(gw[:2], gw[2:]):   # (the bound of the residual block's test)
        scale = float(n * H * W) ** 0.5 * 0.5 + 1.0
        assert torch.allclose(got, want, rtol=1e-5, atol=2.0 ** -20 * scale * max(float(n * H * W) ** 0.5, 1.0))


@pytest.mark.parametrize("n", [1, 15, 16, 17, 200])
@pytest.mark.parametrize("A", [1, 2, 15, 16, 18, 31, 32])   # the head kernel's two 16-row blocks; past them its fallback
@pytest.mark.parametrize("keep_logits", [False, True])
def test_actor_step_samples_as_the_sampling_call_does(n, A, keep_logits):
    """The sample formed by the head kernel is the one impala_gumbel_sample forms from its logits, also
    with ties (noise of few distinct values: the lowest index wins) and with excluded actions."""
    from types import SimpleNamespace
    P = _p()
    net = SimpleNamespace(in_h=20, in_w=18, in_c=4, ch=(16, 32, 32), hidden=256, num_actions=A)
    g = torch.Generator(device="cuda:0").manual_seed(n * 101 + A)
    params = torch.randn(P.impala_param_count(net), generator=g, device="cuda:0") * 0.1
    obs = torch.randint(0, 256, (n, 20, 18, 4), generator=g, device="cuda:0", dtype=torch.int32).to(torch.uint8)
    gum = torch.randint(0, 3, (n, A), generator=g, device="cuda:0").float() * 50.0
    gum[:, A // 2] = -float("inf") if A > 1 else 0.0
    ws = torch.empty(P.impala_workspace_bytes(net, n, P.PREC_BF16, 0) + n * A * 4 + 256, dtype=torch.uint8, device="cuda:0")
    out = []
    for logits in (torch.empty((n, A), device="cuda:0"), torch.empty((n, A), device="cuda:0") if keep_logits else None):
        act = torch.full((n,), -7, dtype=torch.int32, device="cuda:0")
        logp, value = (torch.full((n,), 9.0, device="cuda:0") for _ in range(2))
        P.impala_actor_step(net, P.PREC_BF16, params, obs, n, gum, ws, act, logp, value, logits)
        out.append((act, logp, value, logits))
    act, logp, value, logits = out[0]
    act_ref, logp_ref = torch.empty_like(act), torch.empty_like(logp)
    P.impala_gumbel_sample(n, A, logits, gum, act_ref, logp_ref)
    torch.cuda.synchronize()
    for a, lp, v, _ in out:
        assert torch.equal(a, act_ref)
        assert torch.equal(lp.view(torch.int32), logp_ref.view(torch.int32))
        assert torch.equal(v.view(torch.int32), value.view(torch.int32))


def _network_backward_against_two_halves(ch, n, H, W):
    from types import SimpleNamespace
    P = _p()
    half = n // 2
    net = SimpleNamespace(in_h=H, in_w=W, in_c=4, ch=ch, hidden=256, num_actions=6)
    g = torch.Generator(device="cuda:0").manual_seed(H)
    params = torch.randn(P.impala_param_count(net), generator=g, device="cuda:0") * 0.05
    obs = torch.randint(0, 256, (n, H, W, 4), generator=g, device="cuda:0", dtype=torch.int32).to(torch.uint8)
    dz, dv = torch.randn((n, 6), generator=g, device="cuda:0"), torch.randn(n, generator=g, device="cuda:0")

    def forward(o):
        k = o.shape[0]
        ws = torch.empty(P.impala_workspace_bytes(net, k, P.PREC_BF16, 1), dtype=torch.uint8, device="cuda:0")
        P.impala_cnn_fwd(net, P.PREC_BF16, params, o, None, k, ws, 1, torch.empty((k, 6), device="cuda:0"),
                         torch.empty(k, device="cuda:0"))
        return ws

    whole, want = torch.full_like(params, float("nan")), torch.zeros(params.numel(), dtype=torch.float64, device="cuda:0")
    ws = forward(obs)
    for a in (0, half):
        o, part = obs[a:a + half].contiguous(), torch.full_like(params, float("nan"))
        wh = forward(o)
        # the whole's activations, which both differentiate (the dense layer's sums group by frame count)
        for (name, off, size, _, _), (_, at, hsize, _, _) in zip(P.impala_activation_layout(net, P.PREC_BF16, n),
                                                                 P.impala_activation_layout(net, P.PREC_BF16, half)):
            assert size == 2 * hsize, name
            wh[at:at + hsize] = ws[off + (a // half) * hsize:off + (a // half + 1) * hsize]
        P.impala_cnn_bwd(net, P.PREC_BF16, params, o, None, half, wh, dz[a:a + half].contiguous(),
                         dv[a:a + half].contiguous(), part)
        want += part.double()
    P.impala_cnn_bwd(net, P.PREC_BF16, params, obs, None, n, ws, dz, dv, whole)
    torch.cuda.synchronize()
    # the trunk's gradients are the same bit for bit where the dense input gradient is (its sums over 256 hidden
    # units may round another way: one part in 2^8 of single values), the weight gradients float32 sums
    for name, shape, off in P.impala_param_layout(net):
        w, q = want[off:off + int(np.prod(shape))], whole[off:off + int(np.prod(shape))].double()
        assert (w - q).norm() <= 2.0 ** -10 * w.norm() + 1e-30, (name, float((w - q).norm() / w.norm()))


def test_network_backward_through_the_tile_by_tile_kernel():
    """The whole backward on 1700 frames of 58x68, whose first-stage blocks (29x34) are taken tile by tile and sum
    the launches' partials before them at their start, against the sum over two halves, which walk. A partial of
    the launch before it left out would move its weight gradient by a few percent."""
    _network_backward_against_two_halves((16, 32, 32), 1700, 58, 68)


@pytest.mark.parametrize("ch,n,H,W", [((16, 32, 32), 2, 84, 84), ((16, 32, 32), 24, 84, 84), ((16, 32, 32), 116, 84, 84),
                                      ((16, 32, 32), 250, 84, 84), ((16, 32, 32), 340, 45, 61), ((32, 64, 64), 2, 40, 44),
                                      ((32, 64, 64), 88, 46, 36), ((32, 64, 64), 150, 84, 84), ((16, 16, 32), 400, 84, 84),
                                      # the row counts per walk that those above leave out
                                      ((32, 64, 64), 40, 80, 105), ((16, 16, 32), 148, 29, 110)])
def test_network_backward_of_few_frames(ch, n, H, W):
    """Launches that leave compute units idle, on which the partial sums of the launches before are added up: every
    weight gradient is written, and is the sum of the halves'."""
    _network_backward_against_two_halves(ch, n, H, W)
