"""GPU parity of the glue layers (2x2 max-pool, softmax cross-entropy, SGD with momentum) against
oracle/glue.py, through the C ABI.  Pooling only selects values, so it must agree bit for bit; the loss
and the update compute in fp32 and are held to the fp32 bar (rel-L2 <= 1e-5), bf16 outputs to the bf16 bar."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def env():
    from paper_2112_10065_amd import binding as dp, synth
    from oracle import glue
    import gpu_util as U
    assert torch.cuda.is_available()
    return dp, U, glue, synth


def relu_like(synth, tag, shape, bf16):
    """Post-ReLU activations: about half zeros, so that windows tie."""
    x = np.maximum(synth.normal(tag, shape), 0.0).astype(np.float32)
    return synth.round_bf16(x) if bf16 else x


def upload(U, a, bf16):
    from paper_2112_10065_amd import synth
    return U.bf16_dev(synth.f32_to_bf16_bits(a)) if bf16 else torch.from_numpy(np.ascontiguousarray(a)).to(U.DEV)


POOL_SHAPES = [(2, 12, 10, 64), (1, 5, 7, 16), (3, 4, 4, 8), (2, 6, 9, 12), (1, 1, 6, 8), (2, 7, 1, 5), (1, 2, 2, 1), (2, 28, 28, 512)]


@pytest.mark.parametrize("bf16", [True, False], ids=["bf16", "f32"])
@pytest.mark.parametrize("shape", POOL_SHAPES, ids=["x".join(map(str, s)) for s in POOL_SHAPES])
def test_maxpool_bit_exact(env, shape, bf16):
    dp, U, glue, synth = env
    n, h, w, c = shape
    x = relu_like(synth, f"pool/{shape}", shape, bf16)
    dy = synth.normal(f"pool_dy/{shape}", (n, h // 2, w // 2, c)).astype(np.float32)
    dy = synth.round_bf16(dy) if bf16 else dy
    dt = dp.DP_BF16 if bf16 else dp.DP_F32
    tdt = torch.bfloat16 if bf16 else torch.float32
    xd = upload(U, x, bf16)
    y = torch.full((n, h // 2, w // 2, c), 7.0, dtype=tdt, device=U.DEV)
    dx = torch.full(shape, 7.0, dtype=tdt, device=U.DEV)
    dp.dp_maxpool2x2_fwd(n, h, w, c, dt, xd, y)
    dp.dp_maxpool2x2_bwd(n, h, w, c, dt, xd, upload(U, dy, bf16) if dy.size else None, dx)   # no window: dx is still zeroed
    torch.cuda.synchronize()
    assert np.array_equal(U.to_np(y).astype(np.float64), glue.maxpool2x2_fwd(x))
    assert np.array_equal(U.to_np(dx).astype(np.float64), glue.maxpool2x2_bwd(x, dy))


def test_maxpool_vgg_full_size(env):
    """VGG-16's first pooling layer at per-GPU batch 32 (the size bench.py times): two images against the
    oracle, all of them through properties that hold at any size."""
    dp, U, glue, synth = env
    n, h, w, c = 32, 224, 224, 64
    x = torch.relu(torch.randn((n, h, w, c), device=U.DEV, generator=torch.Generator(device=U.DEV).manual_seed(5))).to(torch.bfloat16)
    dy = torch.randn((n, h // 2, w // 2, c), device=U.DEV, generator=torch.Generator(device=U.DEV).manual_seed(6)).to(torch.bfloat16)
    y = torch.empty((n, h // 2, w // 2, c), dtype=torch.bfloat16, device=U.DEV)
    dx = torch.empty_like(x)
    dp.dp_maxpool2x2_fwd(n, h, w, c, dp.DP_BF16, x, y)
    dp.dp_maxpool2x2_bwd(n, h, w, c, dp.DP_BF16, x, dy, dx)
    torch.cuda.synchronize()
    for i in (0, 31):
        xi, dyi = U.to_np(x[i:i + 1]), U.to_np(dy[i:i + 1])
        assert np.array_equal(U.to_np(y[i:i + 1]).astype(np.float64), glue.maxpool2x2_fwd(xi))
        assert np.array_equal(U.to_np(dx[i:i + 1]).astype(np.float64), glue.maxpool2x2_bwd(xi, dyi))
    # every window hands its gradient to exactly one input, unchanged
    assert int((dx != 0).sum()) == int((dy != 0).sum())
    assert torch.equal(dx.view(n, h // 2, 2, w // 2, 2, c).float().sum(dim=(2, 4)), dy.float())
    assert torch.equal(x.view(n, h // 2, 2, w // 2, 2, c).amax(dim=(2, 4)), y)


@pytest.mark.parametrize("bf16", [True, False], ids=["bf16", "f32"])
@pytest.mark.parametrize("n,classes", [(1, 1000), (32, 1000), (40, 10), (5, 1), (17, 333), (3, 1024), (2, 2500)])
def test_softmax_xent(env, n, classes, bf16):
    dp, U, glue, synth = env
    z = (synth.normal(f"logits/{n}/{classes}", (n, classes)) * 4.0).astype(np.float32)
    z = synth.round_bf16(z) if bf16 else z
    labels = (np.arange(n) * 7919 % classes).astype(np.int32)
    zd = upload(U, z, bf16)
    ld = torch.from_numpy(labels).to(U.DEV)
    loss = torch.zeros(4, dtype=torch.float32, device=U.DEV)
    dz = torch.empty((n, classes), dtype=torch.bfloat16 if bf16 else torch.float32, device=U.DEV)
    dp.dp_softmax_xent(n, classes, dp.DP_BF16 if bf16 else dp.DP_F32, zd, ld, loss, dz)
    torch.cuda.synchronize()
    want_loss, want_dz = glue.softmax_xent(z, labels)
    assert abs(float(loss[0]) - want_loss) <= 1e-5 * max(abs(want_loss), 1e-3)
    if bf16:
        U.assert_bf16_close(U.to_np(dz), want_dz, "dz")
    else:
        rel, mx = U.errs(U.to_np(dz), want_dz)
        assert rel <= U.F32_REL or mx <= 1e-9, f"dz rel_l2={rel:.3e} max_abs={mx:.3e}"
    # loss only (no gradient requested)
    loss2 = torch.zeros(4, dtype=torch.float32, device=U.DEV)
    dp.dp_softmax_xent(n, classes, dp.DP_BF16 if bf16 else dp.DP_F32, zd, ld, loss2, None)
    torch.cuda.synchronize()
    assert float(loss2[0]) == float(loss[0])


@pytest.mark.parametrize("classes", [64, 65, 128, 129, 256, 257, 512, 513, 768, 769])
@pytest.mark.parametrize("bf16", [True, False], ids=["bf16", "f32"])
def test_softmax_xent_at_the_edges_of_the_row_registers(env, classes, bf16):
    test_softmax_xent(env, 18, classes, bf16)


@pytest.mark.parametrize("count", [1, 7, 4096 + 3, 1 << 20, 25088 * 4096])
@pytest.mark.parametrize("with_bf16", [True, False])
def test_sgd_update(env, count, with_bf16):
    dp, U, glue, synth = env
    small = count <= (1 << 20)
    if small:
        w, m, g = (synth.normal(f"sgd/{t}/{count}", (count,)).astype(np.float32) for t in "wmg")
        wd, md, gd = (torch.from_numpy(a.copy()).to(U.DEV) for a in (w, m, g))
    else:   # fc6-sized (bench.py's size): seeded on the device, a slice goes to the oracle
        gen = torch.Generator(device=U.DEV).manual_seed(11)
        wd, md, gd = (torch.randn(count, device=U.DEV, generator=gen) for _ in range(3))
        sl = slice(count - 100003, count)
        w, m, g = (t[sl].cpu().numpy() for t in (wd, md, gd))
    w16 = torch.zeros(count, dtype=torch.bfloat16, device=U.DEV) if with_bf16 else None
    lr, mu = 0.0125, 0.9
    dp.dp_sgd_update(count, lr, mu, gd, md, wd, w16)
    torch.cuda.synchronize()
    want_w, want_m = glue.sgd_momentum(w, m, g, lr, mu)
    got_w, got_m = (wd[sl] if not small else wd).cpu().numpy(), (md[sl] if not small else md).cpu().numpy()
    assert U.errs(got_m, want_m)[0] <= 1e-6 and U.errs(got_w, want_w)[0] <= 1e-6
    assert np.abs(got_w - want_w).max() <= 4e-7 * max(1.0, np.abs(want_w).max())
    if with_bf16:
        assert torch.equal(w16, wd.to(torch.bfloat16))   # round-to-nearest-even copy of the kernel's own fp32 result
