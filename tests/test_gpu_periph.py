"""GPU parity of the digital peripheral kernels (through the C ABI) against their plain definitions."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def xb():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2002_11151_amd import xbar
    xbar.lib()
    return xbar


def dev(a, dtype=np.float32):
    return torch.from_numpy(np.ascontiguousarray(a, dtype=dtype)).cuda()


def close(got, want, tol=2e-6):
    got, want = got.cpu().numpy().astype(np.float64), np.asarray(want, dtype=np.float64)
    assert got.shape == want.shape
    assert np.abs(got - want).max() <= tol * max(1.0, np.abs(want).max())


@pytest.mark.parametrize("B,H,W,C", [(3, 6, 5, 7), (4, 16, 16, 64), (2, 33, 17, 130), (128, 1, 1, 10)])
def test_batchnorm_relu_add(xb, B, H, W, C):
    from oracle import periph
    rng = np.random.default_rng(B + C)
    x = (rng.normal(size=(B, H, W, C)) * 2 + 0.5).astype(np.float32)
    dy = rng.normal(size=(B, H, W, C)).astype(np.float32)
    gamma, beta = rng.uniform(0.5, 1.5, size=C).astype(np.float32), rng.normal(size=C).astype(np.float32)
    y, mean, invstd = xb.bn_fwd(dev(x), dev(gamma), dev(beta), 1e-5)
    yo, mo, io = periph.bn_fwd(x, gamma, beta, 1e-5)
    close(y, yo)
    close(mean, mo)
    close(invstd, io)
    dx, dgamma, dbeta = xb.bn_bwd(dev(x), dev(dy), dev(gamma), mean, invstd)
    dxo, dgo, dbo = periph.bn_bwd(x, dy, gamma, mean.cpu().numpy().astype(np.float64), invstd.cpu().numpy().astype(np.float64))
    close(dx, dxo, 1e-5)
    close(dgamma, dgo, 1e-5)
    close(dbeta, dbo, 1e-5)
    r = xb.relu_fwd(dev(x))
    assert np.array_equal(r.cpu().numpy(), periph.relu_fwd(x).astype(np.float32))
    assert np.array_equal(xb.relu_bwd(r, dev(dy)).cpu().numpy(), periph.relu_bwd(r.cpu().numpy(), dy).astype(np.float32))
    s = xb.sigmoid_fwd(dev(x))
    assert np.abs(s.cpu().numpy() - periph.sigmoid_fwd(x)).max() <= 6e-8                  # half a unit in the last place below 1
    assert np.abs(xb.sigmoid_bwd(s, dev(dy)).cpu().numpy() - periph.sigmoid_bwd(s.cpu().numpy(), dy)).max() <= 1e-7 * np.abs(dy).max()
    assert np.array_equal(xb.add(dev(x), dev(dy)).cpu().numpy(), x + dy)
    p = dev(x.copy())
    xb.sgd(p, dev(dy), 0.1)
    close(p, x.astype(np.float64) - np.float32(0.1).astype(np.float64) * dy, 1e-6)


# Rows that are no quads, one or four of them to a thread: one element, more channels than a block has threads, rows that four do not
# divide; both sides of the line between strips of 16 and of 64 channels
@pytest.mark.parametrize("rows,C", [(1, 1), (2, 257), (7, 259), (1025, 513), (8191, 257), (9001, 257), (53 * 512, 130), (53 * 512 + 1, 130), (53 * 512, 132),
                                    (53 * 512 + 1, 132), (5, 1030)])
def test_normalisation_of_ragged_rows(xb, rows, C):
    from oracle import periph
    rng = np.random.default_rng(rows + C)
    x = (rng.normal(size=(rows, C)) * 2 + 0.5).astype(np.float32)
    dy = rng.normal(size=(rows, C)).astype(np.float32)
    gamma, beta = rng.uniform(0.5, 1.5, size=C).astype(np.float32), rng.normal(size=C).astype(np.float32)
    y, mean, invstd = xb.bn_fwd(dev(x), dev(gamma), dev(beta), 1e-5)
    yo, mo, io = periph.bn_fwd(x, gamma, beta, 1e-5)
    close(mean, mo)
    assert (np.abs(invstd.cpu().numpy() - io) <= 2.0 ** -23 * io).all()
    # mean and 1 / std are stored in single precision, which two rows that lie close to each other multiply by 1 / std
    bound = 2.0 ** -22 * (np.abs(gamma) * io * (np.abs(x) + np.abs(mo)) + np.abs(beta) + np.abs(yo))
    assert (np.abs(y.cpu().numpy() - yo) <= bound).all()
    dx, dgamma, dbeta = xb.bn_bwd(dev(x), dev(dy), dev(gamma), mean, invstd)
    m64, i64 = mean.cpu().numpy().astype(np.float64), invstd.cpu().numpy().astype(np.float64)
    dxo, dgo, dbo = periph.bn_bwd(x, dy, gamma, m64, i64)
    close(dgamma, dgo, 1e-5)
    close(dbeta, dbo, 1e-5)
    bound = 2.0 ** -22 * np.abs(gamma) * i64 * (np.abs(dy) + (np.abs(dbo) + np.abs((x - m64) * i64 * dgo)) / rows)
    assert (np.abs(dx.cpu().numpy() - dxo) <= bound + 1e-30).all()


@pytest.mark.parametrize("B,H,W,C,k,stride,pad", [(2, 9, 8, 5, 3, 2, 1), (3, 8, 8, 64, 2, 2, 0), (1, 7, 7, 3, 3, 1, 1)])
def test_pooling(xb, B, H, W, C, k, stride, pad):
    from oracle import periph
    rng = np.random.default_rng(H + C)
    x = rng.normal(size=(B, H, W, C)).astype(np.float32)
    geom = xb.conv_geom(B, H, W, C, k, k, stride, pad)
    y, arg = xb.maxpool_fwd(dev(x), geom)
    yo, ao = periph.maxpool_fwd(x, k, stride, pad)
    assert np.array_equal(y.cpu().numpy(), yo.astype(np.float32))
    assert np.array_equal(arg.cpu().numpy(), ao)
    d = rng.normal(size=yo.shape).astype(np.float32)
    close(xb.maxpool_bwd(dev(d), arg, geom), periph.maxpool_bwd(d, ao, x.shape))
    a = xb.avgpool_fwd(dev(x))
    close(a, periph.avgpool_fwd(x))
    dg = rng.normal(size=(B, C)).astype(np.float32)
    close(xb.avgpool_bwd(dev(dg), x.shape), periph.avgpool_bwd(dg, x.shape))


# One, four or sixteen threads to an output: positions and outputs on both sides of the lines, outputs that fill no block
@pytest.mark.parametrize("B,positions,C", [(1, 1, 1), (3, 3, 5), (3, 4, 5), (3, 7, 67), (3, 8, 67), (128, 17, 128), (127, 8, 129), (5, 9, 3277), (131, 16, 1000), (131, 9, 1001),
                                           (70000, 2, 3)])
def test_average_pool(xb, B, positions, C):
    from oracle import periph
    x = np.random.default_rng(B + C).normal(size=(B, positions, 1, C)).astype(np.float32)
    close(xb.avgpool_fwd(dev(x)), periph.avgpool_fwd(x))


@pytest.mark.parametrize("B,classes", [(5, 10), (64, 1000), (3, 1)])
def test_softmax_cross_entropy(xb, B, classes):
    from oracle import periph
    rng = np.random.default_rng(classes)
    z = (rng.normal(size=(B, classes)) * 4).astype(np.float32)
    labels = rng.integers(0, classes, size=B).astype(np.int32)
    loss, dz = xb.softmax_xent(dev(z), dev(labels, np.int32), 1.0 / B)
    lo, dzo = periph.softmax_xent(z, labels, np.float32(1.0 / B).astype(np.float64))
    close(loss, lo, 1e-6)
    close(dz, dzo, 1e-6)
    bad = labels.copy()
    bad[0] = classes                                          # unknown class: NaN loss, no fault
    loss, _ = xb.softmax_xent(dev(z), dev(bad, np.int32), 1.0)
    assert np.isnan(loss.cpu().numpy()[0]) and not np.isnan(loss.cpu().numpy()[1:]).any()


@pytest.mark.parametrize("rows,C", [(3, 4), (513, 7), (700, 16), (1100, 36), (2000, 64), (65, 1028), (7, 257), (40000, 64),
                                    (524289, 16), (140001, 61), (131072, 16), (32768, 32), (8192, 64), (12544, 1024), (3136, 2048)])
def test_joined_normalisation_passes(xb, rows, C):
    """Sums and passes at the edges of their strips (16 and 64 channels, quads or not), of 512 rows and of one or four rows per
    thread, and at layers of the networks, against 64 bits; normalisation, addition, ReLU and parameter step in one against the
    single operations, bit for bit."""
    g = torch.Generator(device="cuda").manual_seed(rows + C)
    x, dy, skip = (torch.randn((rows, C), generator=g, device="cuda") for _ in range(3))
    gamma, beta = torch.rand(C, generator=g, device="cuda") + 0.5, torch.randn(C, generator=g, device="cuda")
    y, mean, invstd = xb.bn_fwd(x, gamma, beta)
    X, D = x.double(), dy.double()
    mu, var = X.mean(0), X.var(0, unbiased=False)
    close(mean, mu.cpu().numpy())
    close(invstd, (1 / (var + 1e-5).sqrt()).cpu().numpy(), 1e-6)
    xhat = (X - mean.double()) * invstd.double()
    close(y, (gamma.double() * xhat + beta.double()).cpu().numpy())
    for s in (None, skip):
        y1, mean1, invstd1 = xb.bn_relu_fwd(x, gamma, beta, skip=s)
        want = xb.relu_fwd(y if s is None else xb.add(y, s))
        assert torch.equal(y1, want) and torch.equal(mean1, mean) and torch.equal(invstd1, invstd)
    act = xb.relu_fwd(y)
    assert torch.equal(act, torch.where(y > 0, y, torch.zeros_like(y)))
    assert torch.equal(xb.add_relu_bwd(act, dy, skip), xb.relu_bwd(act, xb.add(dy, skip)))
    for relu in (False, True):
        d = xb.relu_bwd(act, dy) if relu else dy
        assert not relu or torch.equal(d, torch.where(act > 0, dy, torch.zeros_like(dy)))
        want = xb.bn_bwd(x, d, gamma, mean, invstd)
        dg, db = (d.double() * xhat).sum(0), d.double().sum(0)
        scale = rows ** 0.5
        close(want[1] / scale, (dg / scale).cpu().numpy())
        close(want[2] / scale, (db / scale).cpu().numpy())
        dx = gamma.double() * invstd.double() * (d.double() - want[2].double() / rows - xhat * want[1].double() / rows)
        close(want[0], dx.cpu().numpy())
        for lr in (None, 0.1):
            g1, b1 = gamma.clone(), beta.clone()
            got = xb.bn_bwd_sgd(x, dy, g1, b1, mean, invstd, relu=relu, lr=lr)
            assert all(torch.equal(a, b) for a, b in zip(got, want))
            g2, b2 = gamma.clone(), beta.clone()
            if lr is not None:
                xb.sgd(g2, want[1], lr)
                xb.sgd(b2, want[2], lr)
            assert torch.equal(g1, g2) and torch.equal(b1, b2)


def test_joined_passes_keep_nan_and_signs(xb):
    """What is not a number passes no ReLU, forward or backward, and a zero or negative output passes no error."""
    y = torch.tensor([1.0, 0.0, -0.0, -1.0, float("nan"), float("inf"), 2.0], device="cuda")
    a = torch.tensor([1.0, float("nan"), 3.0, 4.0, 5.0, 6.0, float("nan")], device="cuda")
    got, want = xb.add_relu_bwd(y, a, a), xb.relu_bwd(y, xb.add(a, a))
    assert torch.equal(torch.nan_to_num(got, 7.0), torch.nan_to_num(want, 7.0)) and want[5] == 12 and want[4] == 0
    x = torch.randn((64, 8), device="cuda")
    x[3, 2] = float("nan")
    gamma, beta = torch.ones(8, device="cuda"), torch.zeros(8, device="cuda")
    y, mean, invstd = xb.bn_fwd(x, gamma, beta)
    act = xb.bn_relu_fwd(x, gamma, beta)[0]
    assert torch.equal(act, xb.relu_fwd(y)) and not act[:, 2].any()
    dy = torch.randn((64, 8), device="cuda")
    want = xb.bn_bwd(x, xb.relu_bwd(act, dy), gamma, mean, invstd)
    got = xb.bn_bwd_sgd(x, dy, gamma, beta, mean, invstd, relu=True)
    assert all(torch.equal(torch.nan_to_num(u, 7.0), torch.nan_to_num(v, 7.0)) for u, v in zip(got, want))


@pytest.mark.parametrize("kind", ["basic", "bottleneck"])
def test_network_step_joined_or_operation_by_operation(xb, kind):
    """A training step with the joined passes leaves the same losses, weights and parameters as with every operation a call."""
    import workloads
    from paper_2002_11151_amd import resnet_cifar, resnet_imagenet

    class Single:
        def __getattr__(self, name):
            return getattr(xb, name)

    kw = workloads.config_kwargs("resnet20")
    states = []
    for ops in (xb, Single()):
        if kind == "basic":
            net = resnet_cifar.ResNetCifar(kw, batch=3, n_blocks=2, image=12, widths=(8, 16, 20), seed=3)
        else:
            net = resnet_imagenet.ResNetBottleneck(kw, batch=3, image=24, classes=10, blocks=(1, 2), widths=(4, 8), stem=8, seed=3)
        gen = torch.Generator(device="cuda").manual_seed(1)
        images = torch.randn((3, 12, 12, 3) if kind == "basic" else (3, 24, 24, 3), generator=gen, device="cuda")
        labels = torch.tensor([1, 7, 4], dtype=torch.int32, device="cuda")
        net.ops = ops
        net.calibrate(images, labels)
        losses = [net.train_step(images, labels, 0.05).clone() for _ in range(2)]
        norms = [net.stem_bn] + [v for blk in net.blocks for k, v in sorted(blk.items()) if k.startswith("bn")]
        states.append(losses + [layer.W for layer in net.layers] + [t for n in norms for t in (n.gamma, n.beta)])
    assert all(torch.equal(a, b) for a, b in zip(*states))


@pytest.mark.parametrize("B,H,W,C,k,stride,pad", [(2, 9, 8, 8, 3, 2, 1), (1, 7, 7, 4, 3, 1, 1), (2, 11, 6, 20, 2, 3, 1),
                                                  (3, 5, 5, 16, 5, 1, 2)])
def test_pooling_of_quads(xb, B, H, W, C, k, stride, pad):
    """Four channels per thread; windows that overlap, leave gaps between them or hang over the edge."""
    test_pooling(xb, B, H, W, C, k, stride, pad)
