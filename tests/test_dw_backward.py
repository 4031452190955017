"""The backward of a DW + SCC block in one call: the results of its three stages, bit for bit, and the host's checks."""
import ctypes

import pytest
import torch

import paper_2101_00745_amd as S

SHAPES = [(1, 16, 24, 4, 4, 1, 2, 0.5), (3, 32, 40, 9, 7, 2, 4, 0.25), (40, 64, 96, 10, 12, 1, 2, 0.33), (130, 64, 64, 16, 16, 2, 1, 0.5)]


@pytest.mark.gpu
@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("shape", SHAPES)
def test_one_call_is_its_three_stages(shape, dtype):
    N, Cin, Cout, H, W, s, cg, co = shape
    gen = torch.Generator(device="cuda").manual_seed(3)
    x, kdw, w, dy = (torch.randn(*d, generator=gen, device="cuda").to(dtype) for d in
                     ((N, Cin, H, W), (Cin, 3, 3), (Cout, Cin // cg), (N, Cout, (H - 1) // s + 1, (W - 1) // s + 1)))
    z = S.scc_depthwise3x3_forward(x, kdw, s)
    dz, dw = S.scc_backward(z, dy, w, cg, co)
    dx, dk = S.scc_depthwise3x3_backward(x, kdw, dz, s)
    got = S.scc_dw_backward(x, kdw, w, dy, cg, co, s)
    assert all(torch.equal(a, b) and a.dtype == b.dtype for a, b in zip(got, (dx, dk, dw)))


# Maps of strips of 1, 2 and 4 rows, of columns (2x2, 7x7, 6x10) and of single pixels (stride 2 on odd maps, stride 3), one and several
# slices of either filter, fewer than 256 columns, and layers on both sides of the line at 2^23 (columns: 2^22) values of x and z.
# the fused, the shared and the two-pass gradients of the SCC behind them
PAIRED = [(40, 128, 128, 16, 16, 1, 2, 0.5), (128, 128, 512, 32, 32, 1, 2, 0.33), (3, 16, 24, 2, 2, 1, 4, 0.5), (16, 512, 512, 4, 4, 1, 2, 0.5), (16, 1024, 256, 2, 2, 1, 2, 0.5), (5, 48, 40, 7, 7, 1, 4, 0.33), (9, 64, 61, 6, 10, 1, 2, 0.75),
          (20, 64, 96, 13, 9, 2, 2, 0.5), (30, 32, 24, 10, 10, 3, 1, 0.0), (30, 64, 128, 32, 32, 2, 2, 0.5), (128, 32, 64, 32, 32, 1, 2, 0.5),
          (129, 32, 64, 32, 32, 1, 2, 0.5), (167, 256, 256, 7, 7, 1, 4, 0.5), (168, 256, 256, 7, 7, 1, 4, 0.5), (64, 256, 512, 8, 8, 2, 2, 0.5)]


@pytest.mark.gpu
@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("shape", PAIRED)
def test_stages_side_by_side(shape, dtype):
    """The two launches of a block's backward are its three stages, bit for bit, also on the workspace that only the stages
    one after the other run on; and the depthwise filter's gradient is the oracle's."""
    test_one_call_is_its_three_stages(shape, dtype)
    N, Cin, Cout, H, W, s, cg, co = shape
    gen = torch.Generator(device="cuda").manual_seed(3)
    Ho, Wo = (H - 1) // s + 1, (W - 1) // s + 1
    x, kdw, w, dy = (torch.randn(*d, generator=gen, device="cuda").to(dtype) for d in
                     ((N, Cin, H, W), (Cin, 3, 3), (Cout, Cin // cg), (N, Cout, Ho, Wo)))
    dx, dk, dw = S.scc_dw_backward(x, kdw, w, dy, cg, co, s)
    lib, code = S.load(), 0 if dtype == torch.float32 else 1
    shape_c = (N, Cin, Cout, H, W, s, cg, co, code)
    least = int(lib.scc_dw_backward_workspace_bytes(*shape_c))
    assert least <= lib.scc_dw_backward_as_workspace_bytes(*shape_c, 0) <= lib.scc_dw_backward_as_workspace_bytes(*shape_c, 1)
    ws = torch.empty(least, dtype=torch.uint8, device="cuda")
    dx2, dk2, dw2 = torch.empty_like(dx), torch.empty_like(dk), torch.empty_like(dw)
    args = [t.data_ptr() for t in (x, kdw, w, dy, dx2, dk2, dw2)]
    stream = torch.cuda.current_stream().cuda_stream
    assert lib.scc_dw_backward(*args, *shape_c, ws.data_ptr(), least, stream) == 0
    assert torch.equal(dx, dx2) and torch.equal(dk, dk2) and torch.equal(dw, dw2)
    dx3, dk3, dw3 = S.scc._dw_backward(x, kdw, w, dy, cg, co, s, True)       # the same sums, rounded to the weights' type
    assert torch.equal(dx, dx3) and torch.equal(dk.to(dtype), dk3) and torch.equal(dw.to(dtype), dw3)
    if x.numel() <= 1 << 20:
        import numpy as np
        from oracle import scc_oracle as O
        z = S.scc_depthwise3x3_forward(x, kdw, s)
        dz = S.scc_backward(z, dy, w, cg, co)[0]
        ref = O.depthwise3x3_backward(*(t.float().cpu().numpy() for t in (x, kdw, dz)), s)[1]
        assert np.max(np.abs(dk.cpu().numpy() - ref)) <= 2e-5 * np.max(np.abs(ref))     # binary32 sums in both types


def test_narrow_gradients_host_checks():
    lib, p = S.load(), ctypes.c_void_p(0x1000)
    shape = (3, 32, 40, 9, 7, 2, 4, 0.25, 1)
    need = lib.scc_dw_backward_as_workspace_bytes(*shape, 1)
    assert need > lib.scc_dw_backward_workspace_bytes(*shape) > 0
    args = [p] * 7
    assert lib.scc_dw_backward_as(*args, *shape, 1, 0x1000, need - 1, None) == -5 and lib.scc_dw_backward_as(*args, *shape, 1, None, need, None) == -5
    assert lib.scc_dw_backward_as(*args, *shape, 7, 0x1000, need, None) == -4 and lib.scc_dw_backward_as_workspace_bytes(*shape, 7) == 0
    assert lib.scc_dw_backward_as(*args[:-1], None, *shape, 1, 0x1000, need, None) == -1


def test_host_checks():
    lib, p = S.load(), ctypes.c_void_p(0x1000)
    shape = (3, 32, 40, 9, 7, 2, 4, 0.25, 0)
    need = lib.scc_dw_backward_workspace_bytes(*shape)
    assert need >= 2 * 3 * 32 * 5 * 4 * 4
    assert lib.scc_dw_backward(p, p, p, p, p, p, p, *shape, 0x1000, need - 1, None) == -5
    assert lib.scc_dw_backward(p, p, p, p, p, p, p, *shape, None, need, None) == -5
    assert lib.scc_dw_backward(p, p, p, None, p, p, p, *shape, 0x1000, need, None) == -1
    bad = (3, 32, 40, 9, 7, 0, 4, 0.25, 0)
    assert lib.scc_dw_backward(p, p, p, p, p, p, p, *bad, 0x1000, need, None) == -2 and lib.scc_dw_backward_workspace_bytes(*bad) == 0


@pytest.mark.gpu
@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("N,C,s", [(1, 1, 1), (3, 64, 1), (31, 65, 1), (32, 63, 2), (33, 130, 1), (130, 64, 2), (67, 200, 2), (128, 1024, 1), (5, 2000, 2)])
def test_filter_gradient_of_2x2_maps(N, C, s, dtype):
    """A lane per channel: groups of channels whole and partial, samples that fill no, one and several batches of the lanes that
    share them, one and more slices; alone and in a block's backward."""
    gen = torch.Generator(device="cuda").manual_seed(6)
    x, kdw, dz = (torch.randn(*d, generator=gen, device="cuda").to(dtype) for d in ((N, C, 2 * s, 2 * s), (C, 3, 3), (N, C, 2, 2)))
    import numpy as np
    from oracle import scc_oracle as O
    ref_dx, ref_dk = O.depthwise3x3_backward(*(t.float().cpu().numpy() for t in (x, kdw, dz)), s)
    dx, dk = S.scc_depthwise3x3_backward(x, kdw, dz, s)
    assert np.max(np.abs(dk.cpu().numpy() - ref_dk)) <= 2e-6 * np.max(np.abs(ref_dk))     # binary32 sums of 4 N products, as trees
    assert torch.equal(dk, S.scc_depthwise3x3_backward(x, kdw, dz, s, need_dx=False)[1])
    if C % 16 == 0 and N >= 16:
        test_one_call_is_its_three_stages((N, C, 24, 2 * s, 2 * s, s, 2, 0.5), dtype)


@pytest.mark.gpu
@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("N,C,s", [(1024, 7, 1), (1024, 8, 2), (255, 9, 1), (256, 17, 2), (257, 1031, 1), (129, 1024, 2), (1024, 1024, 1), (1024, 1025, 2)])
def test_filter_gradient_of_2x2_maps_of_large_batches(N, C, s, dtype):
    """Eight channels per workgroup, whole and not, and samples that fill one and several batches of its 32 groups of lanes."""
    test_filter_gradient_of_2x2_maps(N, C, s, dtype)


@pytest.mark.gpu
@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("N,C,H,W,s", [(1, 3, 4, 4, 1), (129, 5, 4, 4, 1), (70, 9, 6, 8, 1), (33, 2, 5, 12, 1), (40, 7, 32, 32, 1),
                                       (65, 4, 8, 8, 2), (3, 6, 10, 24, 2), (257, 2, 4, 8, 2)])
def test_depthwise_gradients_in_one_launch_are_those_of_two(N, C, H, W, s, dtype):
    """Strips of 1, 2 and 4 rows, strips per channel below, at and above a workgroup's 256 threads, both strides."""
    gen = torch.Generator(device="cuda").manual_seed(5)
    x, kdw, dz = (torch.randn(*d, generator=gen, device="cuda").to(dtype) for d in
                  ((N, C, H, W), (C, 3, 3), (N, C, (H - 1) // s + 1, (W - 1) // s + 1)))
    dx, dk = S.scc_depthwise3x3_backward(x, kdw, dz, s)
    assert torch.equal(dx, S.scc_depthwise3x3_backward(x, kdw, dz, s, need_dk=False)[0])
    assert torch.equal(dk, S.scc_depthwise3x3_backward(x, kdw, dz, s, need_dx=False)[1])
    import numpy as np
    from oracle import scc_oracle as O
    ref_dx, ref_dk = O.depthwise3x3_backward(*(t.float().cpu().numpy() for t in (x, kdw, dz)), s)
    assert np.max(np.abs(dx.float().cpu().numpy() - ref_dx)) <= (2e-5 if dtype == torch.float32 else 1e-2) * np.max(np.abs(ref_dx))
    assert np.max(np.abs(dk.cpu().numpy() - ref_dk)) <= 2e-5 * np.max(np.abs(ref_dk))


@pytest.mark.gpu
def test_products_of_the_gradient_at_stride_2():
    """A pixel's sum of two or four products: the first is rounded, each that follows is added with one rounding, in the order of the
    rows from below, in every kernel (alone, beside the filter's gradient, in a block's backward)."""
    import numpy as np
    N, C, Ho = 3, 32, 4
    gen = torch.Generator(device="cuda").manual_seed(5)
    x, kdw, dz = (torch.randn(*d, generator=gen, device="cuda") for d in ((N, C, 2 * Ho, 2 * Ho), (C, 3, 3), (N, C, Ho, Ho)))
    g = np.zeros((N, C, Ho + 1, Ho + 1), dtype=np.longdouble)              # rows and columns past the map are zero
    g[:, :, :Ho, :Ho] = dz.cpu().numpy()
    k = kdw.cpu().numpy().astype(np.longdouble).reshape(C, 9, 1, 1)
    a, right, down, both = g[:, :, :-1, :-1], g[:, :, :-1, 1:], g[:, :, 1:, :-1], g[:, :, 1:, 1:]
    one = lambda s: s.astype(np.float32).astype(np.longdouble)             # a binary32 rounding (64 bits hold the exact sum but for ties)
    want = np.empty((N, C, 2 * Ho, 2 * Ho), dtype=np.float32)
    want[:, :, ::2, ::2] = k[:, 4] * a
    want[:, :, ::2, 1::2] = k[:, 5] * a + one(k[:, 3] * right)
    want[:, :, 1::2, ::2] = k[:, 7] * a + one(k[:, 1] * down)
    want[:, :, 1::2, 1::2] = k[:, 8] * a + one(k[:, 6] * right + one(k[:, 2] * down + one(k[:, 0] * both)))
    want = torch.from_numpy(want).cuda()
    assert torch.equal(S.scc_depthwise3x3_backward(x, kdw, dz, 2)[0], want)
    assert torch.equal(S.scc_depthwise3x3_backward(x, kdw, dz, 2, need_dk=False)[0], want)


@pytest.mark.gpu
@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("N,C,H,W", [(17, 1024, 4, 5), (18, 1024, 4, 5), (29, 1030, 2, 6), (30, 1030, 2, 6), (7, 1024, 5, 10), (38, 1024, 4, 5), (200, 1024, 1, 9), (300, 1024, 4, 1),
                                     (9, 1024, 7, 7), (5, 3, 9, 9), (1, 700, 13, 6), (2, 1100, 13, 14)])
def test_filter_gradient_on_columns_or_pixels(N, C, H, W, dtype):
    """On both sides of the line of 350 pixels to a workgroup, in columns of one, two and four rows; maps of one row and of one column."""
    test_depthwise_gradients_in_one_launch_are_those_of_two(N, C, H, W, 1, dtype)
    test_one_call_is_its_three_stages((N, C, 24, H, W, 1, 1, 0.5), dtype)


# paired and not, on either side of the lines: rows of 4 at both strides, columns, pixels, the gather, 2x2 maps
LINES = [(128, 64, 64, 16, 16, 1, 2, 0.5), (129, 64, 64, 16, 16, 1, 2, 0.5), (192, 512, 512, 4, 4, 1, 2, 0.5), (193, 512, 512, 4, 4, 1, 2, 0.5), (83, 256, 256, 7, 7, 1, 8, 0.5),
         (84, 256, 256, 7, 7, 1, 8, 0.5), (125, 256, 256, 7, 7, 1, 8, 0.5), (126, 256, 256, 7, 7, 1, 8, 0.5), (107, 64, 96, 13, 9, 2, 2, 0.5), (108, 64, 96, 13, 9, 2, 2, 0.5), (30, 96, 48, 12, 12, 2, 2, 0.5), (16, 256, 64, 2, 2, 1, 2, 0.5)]


@pytest.mark.gpu
@pytest.mark.parametrize("shift", [(0, 0, 0, 0), (1, 0, 0, 0), (0, 1, 0, 0), (0, 0, 1, 0), (1, 1, 1, 1)])
@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("shape", LINES)
def test_tensors_at_any_address(shape, dtype, shift):
    """x, dy, dx and the weights one element off 16 bytes: other bodies run beside the SCC gradients, with the bits of the stages given
    the same addresses."""
    N, Cin, Cout, H, W, s, cg, co = shape
    Ho, Wo = (H - 1) // s + 1, (W - 1) // s + 1
    gen = torch.Generator(device="cuda").manual_seed(8)

    def at(off, *d, fill=True):
        n = 1
        for v in d:
            n *= v
        t = torch.full((n + 2,), 7.0, dtype=dtype, device="cuda")[off:off + n].view(d)
        return t.copy_(torch.randn(*d, generator=gen, device="cuda")) if fill else t

    x, dy, dx = at(shift[0], N, Cin, H, W), at(shift[1], N, Cout, Ho, Wo), at(shift[2], N, Cin, H, W, fill=False)
    kdw, w = at(shift[3], Cin, 3, 3), at(shift[3], Cout, Cin // cg)
    z = S.scc_depthwise3x3_forward(x, kdw, s)
    dz, dw = S.scc_backward(z, dy, w, cg, co)
    ref_dx, dk = S.scc_depthwise3x3_backward(x, kdw, dz, s, out_dx=at(shift[2], N, Cin, H, W, fill=False))
    lib, code = S.load(), 0 if dtype == torch.float32 else 1
    shape_c = (N, Cin, Cout, H, W, s, cg, co, code)
    need = int(lib.scc_dw_backward_as_workspace_bytes(*shape_c, 0))
    ws = torch.empty(need, dtype=torch.uint8, device="cuda")
    got_k, got_w = torch.empty_like(dk), torch.empty_like(dw)
    args = [t.data_ptr() for t in (x, kdw, w, dy, dx, got_k, got_w)]
    assert lib.scc_dw_backward(*args, *shape_c, ws.data_ptr(), need, torch.cuda.current_stream().cuda_stream) == 0
    assert torch.equal(dx, ref_dx) and torch.equal(got_k, dk) and torch.equal(got_w, dw)


@pytest.mark.gpu
@pytest.mark.parametrize("value", [float("inf"), float("nan")])
@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("N,C,s", [(3, 9, 1), (300, 64, 2), (1024, 20, 1)])
def test_infinity_and_nan_in_2x2_maps(N, C, s, dtype, value):
    """They stay in the filter of their channel, as one sample of many."""
    gen = torch.Generator(device="cuda").manual_seed(9)
    x, kdw, dz = (torch.randn(*d, generator=gen, device="cuda").to(dtype) for d in ((N, C, 2 * s, 2 * s), (C, 3, 3), (N, C, 2, 2)))
    clean = S.scc_depthwise3x3_backward(x, kdw, dz, s)[1]
    for t, at in ((x, (N - 1, C - 2, 0, 0)), (dz, (N // 2, C - 2, 0, 0))):
        kept = t[at].clone()
        t[at] = value
        dk = S.scc_depthwise3x3_backward(x, kdw, dz, s)[1]
        t[at] = kept
        other = torch.arange(C, device="cuda") != C - 2
        assert torch.equal(dk[other], clean[other]) and not bool(torch.isfinite(dk[C - 2, 1, 1]))
