"""The convolution kernels that stage a block of voxels in local memory, at the
edges of their blocks and chunks.

Shapes: blocks cut by the grid in every direction, rows of one voxel, rows
split into pieces, fewer voxels than one tile, last chunks of a few voxels,
chunks that cross slices and batch entries, and rows too wide for the weight
gradient's region (generic kernel).  The forward is compared with the FP64
oracle within the float32 accumulation error K u sum |a_k b_k|, u = 2^-23; the
weight gradient bit for bit with the generic kernel, whose operands, order and
partial sums it shares and which takes inputs off the 16-byte alignment.
"""
import numpy as np
import pytest

from oracle import cnn as ocnn

pytestmark = pytest.mark.gpu

U32 = 2.0 ** -23
_SHAPES = [(1, 1, 1, 1), (2, 3, 1, 2), (3, 5, 7, 11), (1, 13, 33, 12), (1, 9, 11, 47), (1, 2, 3, 200), (2, 6, 5, 64),
           (1, 3, 2, 600), (8, 16, 16, 16)]
_CHANNELS = [(4, 16), (6, 16), (16, 16), (16, 3)]


@pytest.mark.parametrize("ci,co", _CHANNELS)
@pytest.mark.parametrize("shape", _SHAPES, ids=lambda s: "x".join(map(str, s)))
def test_blocks(shape, ci, co):
    import torch
    from paper_1507_06767_amd import cnn
    n, d, h, wd = shape
    nv, c4 = n * d * h * wd, cnn.pad4(ci)
    print(f"\n[case] blocks {shape} {ci}->{co}", flush=True)
    rng = np.random.default_rng(nv + 31 * ci + co)
    x = rng.standard_normal(shape + (ci,)).astype(np.float32)
    w = (rng.standard_normal((co, 27, ci)) * 0.2).astype(np.float32)
    b = (rng.standard_normal(co) * 0.1).astype(np.float32)
    dev = lambda a: torch.tensor(np.ascontiguousarray(a), dtype=torch.float32, device="cuda")
    xp = np.zeros((nv, c4), dtype=np.float32)
    xp[:, :ci] = x.reshape(nv, ci)
    packed = torch.zeros(cnn.lbm_cnn_packed_size(co, ci), dtype=torch.int16, device="cuda")
    assert cnn.lbm_cnn_pack_weights(dev(w), co, ci, 0, packed) == 0
    xd, y = dev(xp), torch.full((nv, cnn.pad4(co)), float("nan"), dtype=torch.float32, device="cuda")
    assert cnn.lbm_cnn_conv3d_forward(xd, n, d, h, wd, ci, packed, co, dev(b), 0, None, y) == 0
    torch.cuda.synchronize()
    got = y.cpu().numpy().astype(np.float64)
    xq, wq = ocnn.bf16_round(x), ocnn.bf16_round(w)
    ref = ocnn.conv3d(xq, wq, b.astype(np.float64)).reshape(nv, co)
    bound = (27 * ci + 1) * U32 * (ocnn.conv3d(np.abs(xq), np.abs(wq)) + np.abs(b)).reshape(nv, co) + 1e-30
    assert (np.abs(got[:, :co] - ref) <= bound).all()
    assert (got[:, co:] == 0).all()

    gz = np.zeros((nv, cnn.pad4(co)), dtype=np.float32)
    gz[:, :co] = rng.standard_normal((nv, co))
    work = [torch.full((cnn.lbm_cnn_wgrad_workspace(n, d, h, wd, ci, co) // 4,), float("nan"), dtype=torch.float32,
                       device="cuda") for _ in range(2)]
    shifted = torch.zeros(nv * c4 + 1, dtype=torch.float32, device="cuda")[1:]
    shifted.copy_(xd.view(-1))
    for a, ws in zip((xd, shifted), work):
        assert cnn.lbm_cnn_conv3d_wgrad_partials(a, dev(gz), n, d, h, wd, ci, co, ws) == 0
    torch.cuda.synchronize()
    a, b = (t.cpu().numpy().view(np.uint32) for t in work)
    # (columns of padding channels hold zeros of either sign)
    zero = lambda v: (v & 0x7fffffff) == 0
    assert ((a == b) | (zero(a) & zero(b))).all()
