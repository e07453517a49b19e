"""The forms of the convolution kernels and the rules that pick them: generic
(any channels), direct (an operand load per tap) and staged in local memory,
in few and in many taps per workgroup, at sizes on either side of the rules."""
import numpy as np
import pytest

from oracle import cnn as ocnn

pytestmark = pytest.mark.gpu

U32 = 2.0 ** -23


@pytest.fixture(scope="module")
def env():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    from paper_1507_06767_amd import cnn
    return torch, cnn


def _dev(torch, a):
    return torch.tensor(np.ascontiguousarray(a), dtype=torch.float32, device="cuda")


def _padded(a, c4):
    out = np.zeros(a.shape[:-1] + (c4,), dtype=np.float32)
    out[..., :a.shape[-1]] = a
    return out


def _shifted(torch, t):
    """The tensor 4 bytes off the 16-byte alignment."""
    s = torch.zeros(t.numel() + 1, dtype=torch.float32, device="cuda")[1:]
    s.copy_(t.reshape(-1))
    return s


def _same(torch, a, b):
    """Equal bits, zeros of either sign alike (columns of padding channels)."""
    return bool(((a.view(torch.int32) == b.view(torch.int32)) | ((a == 0) & (b == 0))).all())


@pytest.mark.parametrize("shape", [(2, 5, 6, 7), (1, 4, 3, 21), (1, 1, 9, 16)], ids=lambda s: "x".join(map(str, s)))
@pytest.mark.parametrize("ci,co", [(20, 16), (32, 32), (32, 1), (128, 5)])
def test_generic_channels(env, shape, ci, co):
    """Channel counts that only the generic kernels take: the forward and the
    masked data gradient (co -> ci channels through ci -> co weights and back)
    within the float32 accumulation error K u sum |a_k b_k|, u = 2^-23."""
    torch, cnn = env
    n, d, h, wd = shape
    nv = n * d * h * wd
    print(f"\n[case] generic {shape} {ci}->{co}", flush=True)
    rng = np.random.default_rng(ci + co + nv)
    x = rng.standard_normal(shape + (ci,)).astype(np.float32)
    w = (rng.standard_normal((co, 27, ci)) * 0.2).astype(np.float32)
    b = (rng.standard_normal(co) * 0.1).astype(np.float32)
    packed = torch.zeros(cnn.lbm_cnn_packed_size(co, ci), dtype=torch.int16, device="cuda")
    flip = torch.zeros(cnn.lbm_cnn_packed_size(ci, co), dtype=torch.int16, device="cuda")
    assert cnn.lbm_cnn_pack_weights(_dev(torch, w), co, ci, 0, packed) == 0
    assert cnn.lbm_cnn_pack_weights(_dev(torch, w), co, ci, 1, flip) == 0
    xq, wq = ocnn.bf16_round(x), ocnn.bf16_round(w)
    ref = ocnn.conv3d(xq, wq, b.astype(np.float64))
    bound = (27 * ci + 1) * U32 * (ocnn.conv3d(np.abs(xq), np.abs(wq)) + np.abs(b)) + 1e-30
    y = torch.full((nv, cnn.pad4(co)), float("nan"), dtype=torch.float32, device="cuda")
    for relu in (0, 1):
        assert cnn.lbm_cnn_conv3d_forward(_dev(torch, _padded(x, cnn.pad4(ci))), n, d, h, wd, ci, packed, co,
                                          _dev(torch, b), relu, None, y) == 0
        got = y.cpu().numpy().astype(np.float64).reshape(shape + (-1,))
        assert (np.abs(got[..., :co] - (ocnn.relu(ref) if relu else ref)) <= bound).all()
        assert (got[..., co:] == 0).all()

    # ci channels of gradient: the layer below has co channels, whose weights
    # are w with the two sides exchanged
    gz = rng.standard_normal(shape + (co,)).astype(np.float32)
    act = rng.standard_normal((nv, cnn.pad4(ci))).astype(np.float32)
    act[::5] = 0.0
    gin = torch.full((nv, cnn.pad4(ci)), float("nan"), dtype=torch.float32, device="cuda")
    assert cnn.lbm_cnn_conv3d_forward(_dev(torch, _padded(gz, cnn.pad4(co))), n, d, h, wd, co, flip, ci, None, 0,
                                      _dev(torch, act), gin) == 0
    gq = ocnn.bf16_round(gz)
    ref = ocnn.conv3d_dgrad(gq, wq).reshape(nv, ci) * (act[:, :ci] > 0)
    bound = 27 * co * U32 * ocnn.conv3d_dgrad(np.abs(gq), np.abs(wq)).reshape(nv, ci) + 1e-30
    assert (np.abs(gin.cpu().numpy()[:, :ci] - ref) <= bound).all()


@pytest.mark.parametrize("channels,shape", [((6, 32, 32, 1), (2, 7, 9, 12)), ((4, 16, 16, 1), (1, 24, 24, 24)),
                                            ((6, 16, 16, 1), (3, 21, 30, 27))])
def test_network_gradients(env, channels, shape):
    """A network with 32-channel layers (generic kernels), and ones of the
    sizes at which the direct and the staged forms take over: loss and
    gradients against the oracle with bfloat16-rounded products.  The bound is
    that of the 16^3 networks: values that round to different sides between
    layers, 5e-3 in relative L2 norm."""
    torch, cnn = env
    from paper_1507_06767_amd.predictor import FlagPredictor
    print(f"\n[case] network {channels} {shape}", flush=True)
    net = FlagPredictor(channels=channels, seed=3)
    rng = np.random.default_rng(9)
    x = rng.standard_normal(shape + (channels[0],)).astype(np.float32)
    t = rng.standard_normal(shape).astype(np.float32)
    loss = net.loss_and_grads(x, t).item()
    params = [(L.w.cpu().numpy().astype(np.float64), L.b.cpu().numpy().astype(np.float64)) for L in net.layers]
    ref_loss, ref = ocnn.loss_and_grads(params, x, t, q=ocnn.bf16_round)
    assert abs(loss - ref_loss) <= 1e-4 * ref_loss
    for L, (rw, rb) in zip(net.layers, ref):
        for got, want in ((L.gw, rw), (L.gb, rb)):
            got = got.cpu().numpy().astype(np.float64)
            assert np.linalg.norm(got - want) < 5e-3 * np.linalg.norm(want)


# voxels on either side of 8,192 and 27,000 (16 channels: taps per workgroup,
# direct and staged), 65,536 (4 and 8 channels: taps per workgroup) and 131,072;
# rows of a multiple of 4 voxels (aligned and shifted inputs take the staged or
# the direct form) and others (staged or generic); chunks that cross slices
# and batch entries, rows too wide for a staged region, grids of short rows
_GRIDS = [(1, 1, 5, 8), (2, 16, 16, 16), (1, 21, 22, 19), (9, 11, 9, 10), (1, 24, 24, 24), (3, 21, 23, 20), (5, 17, 19, 20),
          (2, 37, 31, 29), (3, 29, 31, 28), (4, 32, 32, 32), (40, 4, 4, 4), (2, 16, 16, 200), (1, 3, 2, 600),
          (1, 2, 5, 601)]


@pytest.mark.parametrize("ci,co", [(4, 16), (6, 16), (16, 16), (13, 20), (16, 1)])
@pytest.mark.parametrize("shape", _GRIDS, ids=lambda s: "x".join(map(str, s)))
def test_weight_gradient_forms(env, shape, ci, co):
    """Inputs 4 bytes off the alignment take another form than aligned ones:
    the same partial sums, bit for bit."""
    torch, cnn = env
    n, d, h, wd = shape
    nv = n * d * h * wd
    print(f"\n[case] weight gradient {shape} {ci}->{co}", flush=True)
    g = torch.Generator(device="cuda").manual_seed(nv + ci)
    x = torch.randn((nv, cnn.pad4(ci)), device="cuda", generator=g)
    gz = torch.randn((nv, cnn.pad4(co)), device="cuda", generator=g)
    x[:, ci:] = 0
    gz[:, co:] = 0
    xs, gs = _shifted(torch, x), _shifted(torch, gz)
    p16 = lambda k: (k + 15) // 16 * 16
    used = (nv + 511) // 512 * p16(co) * (p16(27 * cnn.pad4(ci)) + 1)
    got = []
    for a, b in ((x, gz), (xs, gz), (xs, gs)):
        work = torch.full((cnn.lbm_cnn_wgrad_workspace(n, d, h, wd, ci, co) // 4,), float("nan"), device="cuda")
        assert cnn.lbm_cnn_conv3d_wgrad_partials(a, b, n, d, h, wd, ci, co, work) == 0
        got.append(work[:used])
    assert torch.isfinite(got[0]).all()
    for w in got[1:]:
        assert _same(torch, got[0], w)


@pytest.mark.parametrize("ci,co", [(4, 16), (16, 16), (16, 1), (3, 4)])
@pytest.mark.parametrize("shape", _GRIDS, ids=lambda s: "x".join(map(str, s)))
def test_backward_layer_forms(env, shape, ci, co):
    """One launch for a layer's backward gives the bits of the two, with
    aligned and shifted inputs; and the data gradient's one-launch forms those
    of a forward over one batch entry at a time (other forms at other sizes)."""
    torch, cnn = env
    n, d, h, wd = shape
    nv = n * d * h * wd
    i4, o4 = cnn.pad4(ci), cnn.pad4(co)
    print(f"\n[case] backward layer {shape} {ci}->{co}", flush=True)
    g = torch.Generator(device="cuda").manual_seed(nv + ci)
    x = torch.randn((nv, i4), device="cuda", generator=g)
    gz = torch.randn((nv, o4), device="cuda", generator=g)
    x[:, ci:] = 0
    gz[:, co:] = 0
    mask = torch.randn((nv, i4), device="cuda", generator=g)
    w = 0.2 * torch.randn((co, 27, ci), device="cuda", generator=g)
    flip = torch.zeros(cnn.lbm_cnn_packed_size(ci, co), dtype=torch.int16, device="cuda")
    assert cnn.lbm_cnn_pack_weights(w, co, ci, 1, flip) == 0
    p16 = lambda k: (k + 15) // 16 * 16
    used = (nv + 511) // 512 * p16(co) * (p16(27 * i4) + 1)
    nan = lambda m: torch.full((m,), float("nan"), device="cuda")
    size = cnn.lbm_cnn_wgrad_workspace(n, d, h, wd, ci, co) // 4
    ref_w, ref_g, one = nan(size), nan(nv * i4), nan(nv * i4)
    assert cnn.lbm_cnn_conv3d_wgrad_partials(x, gz, n, d, h, wd, ci, co, ref_w) == 0
    assert cnn.lbm_cnn_conv3d_forward(gz, n, d, h, wd, co, flip, ci, None, 0, mask, ref_g) == 0
    for k in range(n):
        part = lambda t, c: t.view(-1)[k * d * h * wd * c:(k + 1) * d * h * wd * c]
        assert cnn.lbm_cnn_conv3d_forward(part(gz, o4), 1, d, h, wd, co, flip, ci, None, 0, part(mask, i4),
                                          part(one, i4)) == 0
    assert torch.isfinite(ref_g).all() and _same(torch, ref_g, one)
    for a in (x, _shifted(torch, x)):
        work, gin = nan(size), nan(nv * i4)
        assert cnn.lbm_cnn_backward_layer(a, gz, n, d, h, wd, ci, co, work, flip, mask, gin) == 0
        assert _same(torch, work[:used], ref_w[:used]) and torch.equal(gin.view(torch.int32), ref_g.view(torch.int32))


def test_forms_of_shifted_and_wide_inputs_are_fast(env):
    """The 16-channel weight gradient of 65,536 voxels off the alignment takes
    at most twice as long as on it, and rows of 256 voxels at most twice as
    long as rows of 64: no fall to the generic kernel, which takes three times
    as long."""
    torch, cnn = env
    stream = torch.cuda.Stream()

    def time(shape, shift):
        n, d, h, wd = shape
        nv = n * d * h * wd
        x, gz = torch.randn(nv * 16, device="cuda"), torch.randn(nv * 16, device="cuda")
        if shift:
            x, gz = _shifted(torch, x), _shifted(torch, gz)
        work = torch.zeros(cnn.lbm_cnn_wgrad_workspace(n, d, h, wd, 16, 16) // 4, device="cuda")
        torch.cuda.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=stream):
            for _ in range(20):
                assert cnn.lbm_cnn_conv3d_wgrad_partials(x, gz, n, d, h, wd, 16, 16, work, stream) == 0
        best = 1e9
        with torch.cuda.stream(stream):
            for _ in range(6):
                a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
                a.record()
                graph.replay()
                b.record()
                b.synchronize()
                best = min(best, a.elapsed_time(b))
        return best

    aligned, shifted, wide = time((1, 16, 64, 64), False), time((1, 16, 64, 64), True), time((1, 16, 16, 256), False)
    print(f"\naligned {aligned * 50:.1f} us, shifted {shifted * 50:.1f}, rows of 256 {wide * 50:.1f}", flush=True)
    assert shifted <= 2 * aligned and wide <= 2 * aligned
