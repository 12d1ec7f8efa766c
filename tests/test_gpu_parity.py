"""GPU-vs-oracle parity through the C ABI: integers bit-exact, fp32 within 1e-5 abs + 1e-5 rel,
bf16 within 1e-2 rel.  Inputs are seeded and synthetic; no expected value comes from the GPU."""
import numpy as np
import pytest
import torch

import oracle
import paper_2404_00509_amd as mae
from paper_2404_00509_amd import synth

from helpers import (ATOL, BF16_RTOL, RTOL, assert_close, assert_close_device, check_grad,
                     check_neutral_outputs,
                     check_prep_against_oracle,
                     gpu_loss, gpu_prep, prep_to_numpy, to_device)

pytestmark = pytest.mark.gpu


def _kw(wl, seed=0, batch_index=0, **extra):
    kw = dict(out_size=wl.out_size, patch=wl.patch,
              num_keep=oracle.num_keep(wl.L, wl.mask_ratio), seed=seed, batch_index=batch_index)
    kw.update(extra)
    return kw


# ------------------------------------------------------------------------------------------------
# whole configurations that the oracle finishes in seconds
# ------------------------------------------------------------------------------------------------
@pytest.mark.parametrize("name", ["c1", "c2"])
def test_prep_small_configs_full(name):
    wl = synth.WORKLOADS[name]
    data = synth.make_images(wl.kind, wl.B, seed=0)
    kw = _kw(wl)
    ref = oracle.prep_batch(*data, **kw)
    buf, _, _ = gpu_prep(*data, **kw)
    assert mae.mae_prep_status(buf.workspace) == 0
    check_prep_against_oracle(prep_to_numpy(buf), ref, what=name)


def test_prep_and_loss_c3_full():
    wl = synth.WORKLOADS["c3"]
    data = synth.make_images(wl.kind, wl.B, seed=0)
    kw = _kw(wl, batch_index=3)
    ref = oracle.prep_batch(*data, **kw)
    buf, _, _ = gpu_prep(*data, **kw)
    check_prep_against_oracle(prep_to_numpy(buf), ref, what="c3")

    # loss: both sides start from the oracle's target and mask
    pred = synth.make_pred(0, wl.B, wl.L, wl.D)
    M = int(ref["mask"].sum())
    assert M == wl.B * (wl.L - kw["num_keep"])
    ref_loss, ref_grad, _ = oracle.normpix_loss(pred, ref["target"], ref["mask"], num_masked=M)
    loss, grad = gpu_loss(torch.from_numpy(pred).cuda(), torch.from_numpy(ref["target"]).cuda(),
                          torch.from_numpy(ref["mask"]).cuda(), num_masked=M)
    assert abs(loss - ref_loss) <= ATOL + RTOL * abs(ref_loss)
    g = grad.cpu().numpy()
    check_grad(g, ref_grad, wl.D, M, what="c3")
    assert np.all(g[ref["mask"] == 0] == 0.0) and not np.signbit(g[ref["mask"] == 0]).any()

    # chained: the GPU's own target and mask feed the GPU loss
    loss2, _ = gpu_loss(torch.from_numpy(pred).cuda(), buf.target, buf.mask, num_masked=M,
                        want_grad=False)
    assert abs(loss2 - ref_loss) <= ATOL + RTOL * abs(ref_loss)


# ------------------------------------------------------------------------------------------------
# full sizes, in the launch configuration the benchmark times: every image against the oracle
# ------------------------------------------------------------------------------------------------
FULL_CHUNK = 256   # images per oracle call: bounds host memory (154 MB per float tensor at c4)


def _full_size(name, bf16):
    wl = synth.WORKLOADS[name]
    data = synth.make_images(wl.kind, wl.B, seed=0)
    kw = _kw(wl, batch_index=1)
    K = kw["num_keep"]
    buf, _, _ = gpu_prep(*data, bf16=bf16, **kw)
    assert mae.mae_prep_status(buf.workspace) == 0

    # predictions are inputs: generated on the device, copied to the oracle chunk by chunk
    gen = torch.Generator(device="cuda").manual_seed(5)
    pred = torch.randn((wl.B, wl.L, wl.D), generator=gen, device="cuda", dtype=torch.float32)
    if bf16:
        pred = pred.to(torch.bfloat16)
    M = wl.B * (wl.L - K)
    loss, grad = gpu_loss(pred, buf.target, buf.mask, num_masked=M)
    unit = float(wl.D) * float(M) / 2.0

    oracle_loss = 0.0
    for lo in range(0, wl.B, FULL_CHUNK):
        hi = min(lo + FULL_CHUNK, wl.B)
        ref = oracle.prep_batch(*data, b_begin=lo, b_end=hi, **kw)
        what = f"{name}[{lo}:{hi}]"
        # integers bit-exact
        for k in ("ids_restore", "ids_keep", "mask"):
            np.testing.assert_array_equal(getattr(buf, k)[lo:hi].cpu().numpy(), ref[k],
                                          err_msg=what + k)
        crop = buf.crop[lo:hi].cpu().numpy()
        np.testing.assert_array_equal(crop[:, :5], ref["crop"], err_msg=what)
        assert np.all(crop[:, 5] == 1)
        # pixels: every element
        assert_close_device(buf.target[lo:hi], ref["target"], what=what + " target")
        assert_close_device(buf.visible[lo:hi], ref["visible"], atol=ATOL,
                            rtol=BF16_RTOL if bf16 else RTOL, what=what + " visible")
        # loss and gradient of the oracle on ITS target: the chunk's share of the batch loss
        # (same divisor M), every gradient element
        part, ref_grad, _ = oracle.normpix_loss(pred[lo:hi].float().cpu().numpy(), ref["target"],
                                                ref["mask"], num_masked=M)
        oracle_loss += part
        assert_close_device(grad[lo:hi], ref_grad, atol=ATOL, rtol=BF16_RTOL if bf16 else RTOL,
                            scale=unit, what=what + " grad")
    assert abs(loss - oracle_loss) <= ATOL + RTOL * abs(oracle_loss), (loss, oracle_loss)

    # properties that hold at any size
    mask = buf.mask
    assert int(mask.sum().item()) == M
    gathered = torch.gather(buf.target, 1,
                            buf.ids_keep.long()[:, :, None].expand(wl.B, K, wl.D))
    if bf16:
        assert torch.equal(gathered.to(torch.bfloat16), buf.visible)
    else:
        assert torch.equal(gathered, buf.visible)
    assert bool((grad[mask == 0] == 0).all())     # visible rows are exactly zero
    # loss of independent N(0,1) predictions against unit-variance targets is close to 2
    assert 1.9 < loss < 2.1


def test_full_size_c4_fp32():
    _full_size("c4", bf16=False)


def test_full_size_c5_bf16_patch14():
    _full_size("c5", bf16=True)


# ------------------------------------------------------------------------------------------------
# edge cases of the input pipeline
# ------------------------------------------------------------------------------------------------
def _pack(imgs):
    sizes = np.array([im.size for im in imgs], np.int64)
    offsets = np.zeros(len(imgs), np.int64)
    offsets[1:] = np.cumsum(sizes)[:-1]
    flat = np.concatenate([im.reshape(-1) for im in imgs]).astype(np.uint8)
    h = np.array([im.shape[0] for im in imgs], np.int32)
    w = np.array([im.shape[1] for im in imgs], np.int32)
    return flat, offsets, h, w


def _random_images(shapes, seed=0):
    rng = np.random.default_rng(seed)
    return [rng.integers(0, 256, size=(h, w, 3), dtype=np.uint8) for h, w in shapes]


@pytest.mark.parametrize("S,p,K", [(112, 16, 12), (224, 14, 64), (256, 16, 64), (64, 32, 1),
                                   (28, 7, 4), (30, 15, 4), (96, 16, 36), (16, 16, 1),
                                   (2, 2, 1), (44, 22, 2)])
def test_prep_shapes_and_tiny_or_large_images(S, p, K):
    # 1x1, one-row, one-column, small and large images (the last ones exceed the staging tile)
    shapes = [(1, 1), (1, 9), (7, 1), (3, 2), (33, 47), (128, 96), (200, 256), (431, 613),
              (700, 300), (90, 1100)]
    data = _pack(_random_images(shapes, seed=S + p))
    kw = dict(out_size=S, patch=p, num_keep=K, seed=9, batch_index=2)
    ref = oracle.prep_batch(*data, **kw)
    buf, _, _ = gpu_prep(*data, **kw)
    check_prep_against_oracle(prep_to_numpy(buf), ref, what=f"S{S}p{p}")
    buf16, _, _ = gpu_prep(*data, bf16=True, **kw)
    check_prep_against_oracle(prep_to_numpy(buf16), ref, bf16=True, what=f"S{S}p{p}bf16")
    # with the staging buffer sized for larger images, rows of patches are split into column
    # parts and wide crops are staged too
    for hint in (500, 1100):
        big, _, _ = gpu_prep(*data, max_image_side=hint, **kw)
        check_prep_against_oracle(prep_to_numpy(big), ref, what=f"S{S}p{p}hint{hint}")


@pytest.mark.parametrize("S,p,K", [(16, 1, 64), (27, 3, 20), (72, 9, 64), (62, 31, 3), (225, 15, 45),
                                   # both sides of the line between the two kernels
                                   (48, 3, 200), (84, 7, 36), (75, 5, 64), (126, 9, 50),
                                   (124, 31, 4), (93, 31, 3), (19, 19, 1)])
@pytest.mark.parametrize("want_target", [True, False])
def test_prep_odd_patch_sizes(S, p, K, want_target):
    """A pixel per lane: patches of one pixel, of just over one wavefront (81), of 961 pixels; staged,
    split into column parts and from global memory; with and without a target; and a pixel per
    thread where the images are several times as large as the output."""
    shapes = [(1, 1), (5, 300), (130, 97), (256, 200), (431, 613), (90, 1100)]
    data = _pack(_random_images(shapes, seed=S + p))
    kw = dict(out_size=S, patch=p, num_keep=K, seed=9, batch_index=2)
    ref = oracle.prep_batch(*data, **kw)
    dev = to_device(*data)
    for bf16, hint in ((False, 256), (True, 256), (False, 700), (True, 128)):
        desc = mae.make_prep_desc(*dev, max_image_side=hint,
                                  out_dtype=mae.MAE_BF16 if bf16 else mae.MAE_F32, **kw)
        buf = mae.alloc_prep_buffers(desc, want_target=want_target)
        buf.visible.fill_(float("nan"))
        if want_target:
            buf.target.fill_(float("nan"))
        mae.mae_prep_batch(desc, buf.visible, buf.mask, buf.ids_restore, buf.ids_keep, buf.target,
                           buf.crop, buf.workspace)
        assert_close(buf.visible.float().cpu().numpy(), ref["visible"],
                     rtol=BF16_RTOL if bf16 else RTOL, what=f"visible p{p} hint{hint}")
        if want_target:
            assert_close(buf.target.cpu().numpy(), ref["target"], what=f"target p{p} hint{hint}")


def test_prep_odd_patch_with_more_work_items_than_one_launch_takes():
    """262,160 samples of 16 x 16 patches of 31 x 31 pixels would be 2^32 threads of the staged kernel
    and more; the samples equal those of small calls."""
    B, S, p = 262160, 496, 31
    images, offsets, heights, widths = to_device(*_pack(_random_images([(9, 7)], seed=3)))
    src = (images, offsets.expand(B).contiguous(), heights.expand(B).contiguous(),
           widths.expand(B).contiguous())
    kw = dict(out_size=S, patch=p, num_keep=1, seed=10, out_dtype=mae.MAE_BF16)
    desc = mae.make_prep_desc(*src, **kw)
    buf = mae.alloc_prep_buffers(desc, want_target=False)
    mae.mae_prep_batch(desc, buf.visible, buf.mask, buf.ids_restore, buf.ids_keep, None, buf.crop,
                       buf.workspace)
    for b in (0, 1, B // 2, B - 1):
        one = mae.make_prep_desc(images, offsets, heights, widths, sample_base=b, **kw)
        small = mae.alloc_prep_buffers(one, want_target=False)
        mae.mae_prep_batch(one, small.visible, small.mask, small.ids_restore, small.ids_keep, None,
                           small.crop, small.workspace)
        assert torch.equal(buf.visible[b], small.visible[0])
        assert torch.equal(buf.ids_restore[b], small.ids_restore[0])
        assert torch.equal(buf.crop[b], small.crop[0])


def test_prep_single_image_and_keep_all():
    data = _pack(_random_images([(77, 91)]))
    for K in (1, 49):
        kw = dict(out_size=112, patch=16, num_keep=K, seed=1)
        ref = oracle.prep_batch(*data, **kw)
        buf, _, _ = gpu_prep(*data, **kw)
        check_prep_against_oracle(prep_to_numpy(buf), ref, what=f"K{K}")


def test_prep_identity_crop_and_flip_extremes():
    S, p = 64, 16
    imgs = _random_images([(S, S)] * 4, seed=4)
    data = _pack(imgs)
    mean = np.array(mae.IMAGENET_MEAN, np.float32).astype(np.float64)
    std = np.array(mae.IMAGENET_STD, np.float32).astype(np.float64)
    for flip_p in (0.0, 1.0):
        kw = dict(out_size=S, patch=p, num_keep=4, scale=(1.0, 1.0), ratio=(1.0, 1.0),
                  flip_p=flip_p)
        buf, _, _ = gpu_prep(*data, **kw)
        got = prep_to_numpy(buf)
        assert np.all(got["crop"][:, :4] == [0, 0, S, S]) and np.all(got["crop"][:, 4] == flip_p)
        for b, im in enumerate(imgs):
            src = im[:, ::-1] if flip_p else im
            norm = (src.astype(np.float64) / 255.0 - mean) / std
            want = norm.reshape(4, p, 4, p, 3).transpose(0, 2, 1, 3, 4).reshape(16, 768)
            assert_close(got["target"][b], want, what="identity crop")
        check_prep_against_oracle(got, oracle.prep_batch(*data, **kw), what="identity")


@pytest.mark.parametrize("bits", [1, 2, 5, 31])
def test_prep_noise_ties_keep_index_order(bits):
    data = _pack(_random_images([(40, 40)] * 16, seed=2))
    for S, p, K in ((112, 16, 12), (224, 14, 64), (160, 16, 25)):
        kw = dict(out_size=S, patch=p, num_keep=K, noise_bits=bits, seed=3, batch_index=8)
        ref = oracle.prep_batch(*data, want_target=False, want_visible=False, **kw)
        buf, _, _ = gpu_prep(*data, **kw)
        got = prep_to_numpy(buf)
        for k in ("ids_restore", "ids_keep", "mask"):
            np.testing.assert_array_equal(got[k], ref[k])


def test_prep_mask_ratios_of_the_progressive_schemes():
    data = _pack(_random_images([(60, 70)] * 8, seed=6))
    for S in (160, 192, 224):
        L = (S // 16) ** 2
        for m in (0.5, 0.66, 0.75, 0.8, 0.85):
            K = mae.mae_num_keep(L, m)
            assert K == oracle.num_keep(L, m)
            kw = dict(out_size=S, patch=16, num_keep=K, seed=12, batch_index=int(m * 100))
            ref = oracle.prep_batch(*data, want_target=False, want_visible=False, **kw)
            buf, _, _ = gpu_prep(*data, want_target=False, **kw)
            got = prep_to_numpy(buf)
            for k in ("ids_restore", "ids_keep", "mask", ):
                np.testing.assert_array_equal(got[k], ref[k])
            np.testing.assert_array_equal(got["crop"][:, :5], ref["crop"])


def test_prep_fallback_box_on_elongated_images():
    # very elongated images reject all ten proposals and take the centred fallback
    shapes = [(20, 400), (400, 20), (10, 300), (512, 30), (64, 64)]
    data = _pack(_random_images(shapes, seed=8))
    kw = dict(out_size=32, patch=16, num_keep=2, scale=(0.9, 1.0), seed=2)
    used = [oracle.rrc_params(h, w, (0.9, 1.0), (0.75, 4 / 3), 2, 0, b)[1]
            for b, (h, w) in enumerate(shapes)]
    assert used[:4] == [11, 11, 11, 11]
    ref = oracle.prep_batch(*data, **kw)
    buf, _, _ = gpu_prep(*data, **kw)
    check_prep_against_oracle(prep_to_numpy(buf), ref, what="fallback")


def test_prep_is_reproducible_and_keyed_by_batch_and_sample_base():
    wl = synth.WORKLOADS["c1"]
    data = synth.make_images(wl.kind, 32, seed=1)
    kw = _kw(wl, seed=5, batch_index=7)
    a, _, dimg = gpu_prep(*data, **kw)
    b, _, _ = gpu_prep(*data, device_inputs=dimg, **kw)
    for k in ("visible", "mask", "ids_restore", "ids_keep", "target", "crop"):
        assert torch.equal(getattr(a, k), getattr(b, k)), k
    c, _, _ = gpu_prep(*data, device_inputs=dimg, **{**kw, "batch_index": 8})
    assert not torch.equal(a.ids_restore, c.ids_restore)
    assert not torch.equal(a.crop, c.crop)
    # a shard of the batch (samples 20..31 with sample_base 20) equals that slice of the batch
    images, offsets, heights, widths = data
    shard = (images, offsets[20:].copy(), heights[20:].copy(), widths[20:].copy())
    s, _, _ = gpu_prep(*shard, sample_base=20, **kw)
    for k in ("visible", "mask", "ids_restore", "ids_keep", "target", "crop"):
        assert torch.equal(getattr(s, k), getattr(a, k)[20:]), k


@pytest.mark.parametrize("patch,bf16,aug", [(16, False, 0), (16, True, 0), (5, False, 0),
                                            (5, True, 0), (8, False, 1), (8, False, 2)])
def test_prep_gives_unreadable_samples_neutral_outputs(patch, bf16, aug):
    """Geometry is checked on the device; a sample that fails takes no part in the batch (every
    output defined, as the oracle defines it) and its neighbours are unaffected."""
    imgs = _random_images([(30, 30)] * 6, seed=3)
    images, offsets, heights, widths = _pack(imgs)
    heights = heights.copy()
    widths = widths.copy()
    offsets = offsets.copy()
    heights[1] = 0                       # empty image
    widths[2] = 40000                    # wider than supported
    offsets[3] = images.size - 10        # runs past the end of the buffer
    offsets[4] = -3                      # negative offset
    S = 40 if patch != 16 else 32
    L = (S // patch) ** 2
    kw = dict(out_size=S, patch=patch, num_keep=max(1, L // 4), seed=1, aug_mode=aug)
    buf, _, _ = gpu_prep(images, offsets, heights, widths, bf16=bf16, **kw)
    assert mae.mae_prep_status(buf.workspace) == 4
    got = prep_to_numpy(buf)
    assert list(got["crop"][:, 5]) == [1, 0, 0, 0, 0, 1]
    ref = oracle.prep_batch(images, offsets, heights, widths, **kw)
    assert list(ref["valid"]) == [1, 0, 0, 0, 0, 1]
    got["crop"][:, 5] = 1   # the flags were compared above
    check_prep_against_oracle(got, ref, bf16=bf16, what="unreadable samples")
    for b in (1, 2, 3, 4):
        check_neutral_outputs(buf, b)


def test_loss_divisor_counted_on_the_device_leaves_unreadable_samples_out():
    """num_masked = 0: the divisor is the number of masked patches that exist.  A batch with two
    unreadable samples gives the loss and the gradient of the readable ones alone, through both
    forms of the loss call and the one without a workspace."""
    wl = synth.WORKLOADS["c1"]
    B = 10
    images, offsets, heights, widths = synth.make_images(wl.kind, B, seed=4)
    heights = heights.copy()
    offsets = offsets.copy()
    heights[2] = -5
    offsets[7] = images.size
    K = oracle.num_keep(wl.L, wl.mask_ratio)
    kw = dict(out_size=wl.out_size, patch=wl.patch, num_keep=K, seed=3, batch_index=1)
    ref = oracle.prep_batch(images, offsets, heights, widths, **kw)
    pred_host = synth.make_pred(6, B, wl.L, wl.D)
    M = int(ref["mask"].sum())
    assert M == (B - 2) * (wl.L - K)
    ref_loss, ref_grad, _ = oracle.normpix_loss(pred_host, ref["target"], ref["mask"])
    buf, desc, _ = gpu_prep(images, offsets, heights, widths, **kw)
    pred = torch.from_numpy(pred_host).cuda()
    results = {}
    ldesc = mae.make_loss_desc(pred, buf.target, buf.mask, num_masked=0)
    ws = torch.empty(mae.mae_loss_workspace_bytes(ldesc), dtype=torch.uint8, device="cuda")
    for name in ("workspace", "static", "from_images"):
        loss = torch.full((1,), float("nan"), device="cuda")
        grad = torch.full_like(pred, float("nan"))
        if name == "workspace":
            mae.mae_normpix_loss(ldesc, loss, grad, ws)
        elif name == "static":
            mae.mae_normpix_loss_static(ldesc, loss, grad)
        else:
            fdesc = mae.make_loss_desc(pred, None, buf.mask, num_masked=0)
            fws = torch.empty(mae.mae_loss_from_images_workspace_bytes(desc, fdesc),
                              dtype=torch.uint8, device="cuda")
            mae.mae_normpix_loss_from_images(desc, buf.workspace, fdesc, loss, grad, fws)
        torch.cuda.synchronize()
        results[name] = (loss.item(), grad.cpu().numpy())
    for name, (loss, grad) in results.items():
        assert abs(loss - ref_loss) <= ATOL + RTOL * abs(ref_loss), name
        check_grad(grad, ref_grad, wl.D, M, what=name)
        assert not grad[[2, 7]].any(), name
    # nothing masked at all: loss 0, gradient 0, no NaN
    none = torch.zeros_like(buf.mask)
    ldesc = mae.make_loss_desc(pred, buf.target, none, num_masked=0)
    loss = torch.full((1,), float("nan"), device="cuda")
    grad = torch.full_like(pred, float("nan"))
    mae.mae_normpix_loss(ldesc, loss, grad, ws)
    torch.cuda.synchronize()
    assert loss.item() == 0.0 and not grad.any()


# ------------------------------------------------------------------------------------------------
# edge cases of the loss
# ------------------------------------------------------------------------------------------------
def _loss_case(B, L, D, seed, mask_mode="random", bf16=False, grad_scale=1.0, eps=1e-6,
               num_masked=None):
    rng = np.random.default_rng(seed)
    target = (rng.standard_normal((B, L, D)) * rng.uniform(0.2, 3.0, (B, L, 1))
              + rng.uniform(-2, 2, (B, L, 1))).astype(np.float32)
    pred = rng.standard_normal((B, L, D)).astype(np.float32)
    if bf16:
        pred = torch.from_numpy(pred).to(torch.bfloat16).float().numpy()
    if mask_mode == "random":
        mask = (rng.random((B, L)) < 0.75).astype(np.uint8)
        mask[0, 0] = 1
    elif mask_mode == "ones":
        mask = np.ones((B, L), np.uint8)
    elif mask_mode == "single":
        mask = np.zeros((B, L), np.uint8)
        mask[B - 1, L - 1] = 1
    else:
        mask = np.zeros((B, L), np.uint8)
    M = int(mask.sum()) if num_masked is None else num_masked
    ref_loss, ref_grad, _ = oracle.normpix_loss(pred, target, mask, num_masked=M, eps=eps,
                                                grad_scale=grad_scale)
    tp = torch.from_numpy(pred).cuda()
    if bf16:
        tp = tp.to(torch.bfloat16)
    loss, grad = gpu_loss(tp, torch.from_numpy(target).cuda(), torch.from_numpy(mask).cuda(),
                          num_masked=M, eps=eps, grad_scale=grad_scale)
    assert abs(loss - ref_loss) <= ATOL + RTOL * abs(ref_loss), (loss, ref_loss)
    check_grad(grad.float().cpu().numpy(), ref_grad, D, M, grad_scale=grad_scale, bf16=bf16,
               what=f"B{B}L{L}D{D}")
    loss_only, none = gpu_loss(tp, torch.from_numpy(target).cuda(), torch.from_numpy(mask).cuda(),
                               num_masked=M, eps=eps, grad_scale=grad_scale, want_grad=False)
    assert none is None and loss_only == loss


@pytest.mark.parametrize("B,L,D", [(1, 1, 12), (3, 5, 768), (2, 49, 588), (5, 7, 256),
                                   (2, 3, 3072), (1, 9, 1024), (2, 4, 1536), (3, 3, 2048),
                                   (2, 5, 147), (1, 6, 2), (2, 3, 2700), (7, 196, 768),
                                   # no multiple of four: one to three values in the last group, the
                                   # last group alone in its lane's run, every count of groups
                                   # (and the shortest of them, a value per lane)
                                   (3, 5, 3), (4, 9, 5), (3, 7, 27), (5, 5, 63), (3, 9, 65),
                                   (3, 9, 95), (3, 9, 97), (5, 9, 257), (3, 7, 675), (2, 3, 1023), (2, 3, 1025),
                                   (2, 3, 1587), (2, 3, 2046), (1, 3, 2883), (2, 2, 3071)])
@pytest.mark.parametrize("bf16", [False, True])
def test_loss_shapes(B, L, D, bf16):
    _loss_case(B, L, D, seed=B * 1000 + L * 10 + D, bf16=bf16)


@pytest.mark.parametrize("mode", ["ones", "single", "zeros"])
def test_loss_mask_extremes(mode):
    _loss_case(3, 11, 768, seed=1, mask_mode=mode, num_masked=1 if mode == "zeros" else None)


def test_loss_scale_eps_and_constant_rows():
    _loss_case(2, 9, 768, seed=2, grad_scale=-3.5, eps=1e-3, num_masked=1000)
    rng = np.random.default_rng(0)
    B, L, D = 2, 4, 768
    target = rng.standard_normal((B, L, D)).astype(np.float32)
    target[0, 1] = 0.25                     # constant row: variance zero, normalised row zero
    pred = rng.standard_normal((B, L, D)).astype(np.float32)
    mask = np.ones((B, L), np.uint8)
    ref_loss, ref_grad, _ = oracle.normpix_loss(pred, target, mask, num_masked=8)
    loss, grad = gpu_loss(torch.from_numpy(pred).cuda(), torch.from_numpy(target).cuda(),
                          torch.from_numpy(mask).cuda(), num_masked=8)
    assert np.isfinite(loss) and abs(loss - ref_loss) <= ATOL + RTOL * abs(ref_loss)
    check_grad(grad.cpu().numpy(), ref_grad, D, 8, what="constant row")


def test_loss_zero_for_exact_prediction_and_reproducible():
    rng = np.random.default_rng(4)
    B, L, D = 4, 16, 768
    target = rng.standard_normal((B, L, D)).astype(np.float32)
    mask = (rng.random((B, L)) < 0.75).astype(np.uint8)
    M = int(mask.sum())
    _, _, that = oracle.normpix_loss(target, target, mask, num_masked=M, want_that=True)
    pred = that.astype(np.float32)
    args = (torch.from_numpy(pred).cuda(), torch.from_numpy(target).cuda(),
            torch.from_numpy(mask).cuda())
    loss, grad = gpu_loss(*args, num_masked=M)
    assert 0.0 <= loss < 1e-10
    assert float(grad.abs().max().item()) * D * M < 1e-4
    loss2, grad2 = gpu_loss(*args, num_masked=M)
    assert loss2 == loss and torch.equal(grad, grad2)


# ------------------------------------------------------------------------------------------------
# buffer-edge and stream behaviour
# ------------------------------------------------------------------------------------------------
# Crops several times as large as the output: only the rows that are tapped are staged, in an unaligned
# buffer without slack, with outputs of both types and with the augmentations.
@pytest.mark.parametrize("S,p,aug", [(96, 16, 0), (96, 32, 0), (100, 20, 0), (32, 2, 0), (60, 12, 0), (96, 16, 1),
                                     (64, 32, 1), (60, 6, 2), (96, 16, 2)])
def test_prep_of_crops_of_which_only_the_tapped_rows_are_staged(S, p, aug):
    flat, offsets, h, w = synth.make_images("gradient500", 8, seed=70 + S + p)
    L = (S // p) ** 2
    for shift in (0, 3):
        store = torch.zeros(flat.size + shift, dtype=torch.uint8, device="cuda")
        store[shift:] = torch.from_numpy(flat).cuda()
        dimg = (store[shift:], torch.from_numpy(offsets).cuda(), torch.from_numpy(h).cuda(),
                torch.from_numpy(w).cuda())
        kw = dict(out_size=S, patch=p, num_keep=max(1, L // 2), scale=(0.02, 1.0), seed=7 + shift, aug_mode=aug)
        ref = oracle.prep_batch(flat, offsets, h, w, **kw)
        for bf16 in (False, True):
            buf, _, _ = gpu_prep(flat, offsets, h, w, bf16=bf16, device_inputs=dimg, max_image_side=500, **kw)
            check_prep_against_oracle(prep_to_numpy(buf), ref, bf16=bf16, what=f"S{S} p{p} aug {aug}")


# ... and crops that tap nearly all of the rows between the first and the last tapped one, which are staged whole
# up to a quarter more rows than 2 p where that costs no workgroup of a compute unit (or, for the outputs of a batch
# of two rounds of workgroups or fewer, always): on either side of these lines.
@pytest.mark.parametrize("S,p,side,aug", [(224, 16, 500, 0), (240, 16, 500, 0), (112, 16, 256, 0), (112, 14, 256, 0),
                                          (112, 8, 256, 0), (224, 16, 500, 1), (120, 20, 256, 1), (112, 14, 256, 1),
                                          (224, 16, 500, 2), (120, 20, 256, 2), (224, 28, 500, 2)])
def test_prep_of_crops_just_over_twice_the_output(S, p, side, aug):
    data = synth.make_images("gradient500" if side == 500 else "gradient", 6, seed=90 + S + p)
    L = (S // p) ** 2
    kw = dict(out_size=S, patch=p, num_keep=max(1, L // 2), scale=(0.8, 1.0), seed=9, aug_mode=aug)
    assert max(data[2].max(), data[3].max()) == side
    ref = oracle.prep_batch(*data, **kw)
    for bf16 in (False, True):
        buf, _, _ = gpu_prep(*data, bf16=bf16, max_image_side=side, **kw)
        check_prep_against_oracle(prep_to_numpy(buf), ref, bf16=bf16, what=f"S{S} p{p} side {side} aug {aug}")


@pytest.mark.parametrize("shift", [1, 2, 3])
def test_prep_image_buffer_with_unaligned_base_and_tight_end(shift):
    # the staging loads are 4-byte aligned 16-byte reads; with an unaligned base pointer and no
    # slack after the last image, the first and last bytes must come through the guarded path
    shapes = [(40, 52), (64, 64), (33, 47), (80, 61)]
    imgs = _random_images(shapes, seed=shift)
    flat, offsets, h, w = _pack(imgs)
    store = torch.zeros(flat.size + shift, dtype=torch.uint8, device="cuda")
    store[shift:] = torch.from_numpy(flat).cuda()
    dimg = (store[shift:], torch.from_numpy(offsets).cuda(), torch.from_numpy(h).cuda(),
            torch.from_numpy(w).cuda())
    assert dimg[0].data_ptr() % 4 == shift
    for scale in ((1.0, 1.0), (0.2, 1.0)):
        kw = dict(out_size=32, patch=16, num_keep=2, scale=scale, ratio=(1.0, 1.0), seed=shift)
        ref = oracle.prep_batch(flat, offsets, h, w, **kw)
        buf, _, _ = gpu_prep(flat, offsets, h, w, device_inputs=dimg, **kw)
        check_prep_against_oracle(prep_to_numpy(buf), ref, what=f"shift{shift}")


def test_path_on_a_side_stream_and_in_a_captured_graph():
    wl = synth.WORKLOADS["c1"]
    data = synth.make_images(wl.kind, 32, seed=2)
    kw = _kw(wl, seed=1, batch_index=4)
    ref = oracle.prep_batch(*data, **kw)
    K, M = kw["num_keep"], 32 * (wl.L - kw["num_keep"])
    pred_host = synth.make_pred(3, 32, wl.L, wl.D)
    ref_loss, ref_grad, _ = oracle.normpix_loss(pred_host, ref["target"], ref["mask"],
                                                num_masked=M)
    dimg = to_device(*data)
    pred = torch.from_numpy(pred_host).cuda()
    desc = mae.make_prep_desc(*dimg, **kw)
    buf = mae.alloc_prep_buffers(desc)
    ldesc = mae.make_loss_desc(pred, buf.target, buf.mask, num_masked=M)
    lws = torch.empty(max(mae.mae_loss_workspace_bytes(ldesc), 256), dtype=torch.uint8,
                      device="cuda")
    loss = torch.zeros(1, device="cuda")
    grad = torch.empty_like(pred)

    def step(stream):
        mae.mae_prep_batch(desc, buf.visible, buf.mask, buf.ids_restore, buf.ids_keep, buf.target,
                           buf.crop, buf.workspace, stream=stream)
        mae.mae_normpix_loss(ldesc, loss, grad, lws, stream=stream)

    def check(what):
        torch.cuda.synchronize()
        check_prep_against_oracle(prep_to_numpy(buf), ref, what=what)
        assert abs(loss.item() - ref_loss) <= ATOL + RTOL * abs(ref_loss), what
        check_grad(grad.cpu().numpy(), ref_grad, wl.D, M, what=what)

    def wipe():
        for t in (buf.visible, buf.target, grad):
            t.fill_(float("nan"))
        buf.ids_restore.fill_(-1)
        loss.fill_(-1.0)
        torch.cuda.synchronize()

    side = torch.cuda.Stream()
    wipe()
    with torch.cuda.stream(side):
        step(side)
    side.synchronize()
    check("side stream")

    # the calls enqueue only kernels (no memset, no copy, no sync), so they can be captured;
    # every replay is checked against the oracle with eager work in between
    graph = torch.cuda.CUDAGraph()
    wipe()
    with torch.cuda.graph(graph):
        step(torch.cuda.current_stream())
    for replay in range(3):
        wipe()
        graph.replay()
        check(f"graph replay {replay}")
        buf.target.mul_(1.0)          # eager work between replays
        torch.cuda.synchronize()


def test_binding_rejects_tensors_it_would_misread():
    """dtype, contiguity and size are checked before a pointer reaches the library."""
    imgs = _random_images([(30, 30)] * 2, seed=5)
    images, offsets, heights, widths = _pack(imgs)
    dev = to_device(images, offsets, heights, widths)
    kw = dict(out_size=32, patch=16, num_keep=1)
    with pytest.raises(TypeError, match="dtype"):
        mae.make_prep_desc(dev[0], dev[1].int(), dev[2], dev[3], **kw)
    with pytest.raises(TypeError, match="dtype"):
        mae.make_prep_desc(dev[0].float(), dev[1], dev[2], dev[3], **kw)
    desc = mae.make_prep_desc(*dev, **kw)
    buf = mae.alloc_prep_buffers(desc)
    with pytest.raises(TypeError, match="dtype"):          # bf16 tokens asked for, fp32 given
        bad = mae.make_prep_desc(*dev, out_dtype=mae.MAE_BF16, **kw)
        mae.mae_prep_batch(bad, buf.visible, buf.mask, buf.ids_restore, buf.ids_keep, buf.target,
                           buf.crop, buf.workspace)
    with pytest.raises(ValueError, match="elements"):       # target too small
        mae.mae_prep_batch(desc, buf.visible, buf.mask, buf.ids_restore, buf.ids_keep,
                           buf.target[:1], buf.crop, buf.workspace)
    pred = torch.zeros((2, 4, 768), device="cuda")
    mask = torch.ones((2, 4), dtype=torch.uint8, device="cuda")
    with pytest.raises(TypeError, match="dtype"):           # fp16 is not a prediction type
        mae.make_loss_desc(pred.half(), pred, mask, num_masked=8)
    with pytest.raises(ValueError, match="contiguous"):
        mae.make_loss_desc(pred.transpose(0, 1), pred, mask, num_masked=8)
    ldesc = mae.make_loss_desc(pred, pred, mask, num_masked=8)
    with pytest.raises(TypeError, match="dtype"):           # gradient of another type
        mae.mae_normpix_loss(ldesc, torch.zeros(1, device="cuda"), pred.to(torch.bfloat16),
                             torch.empty(4096, dtype=torch.uint8, device="cuda"))
    with pytest.raises(TypeError, match="dtype"):           # fp32 tokens into the bf16 embedding
        mae.make_embed_desc(pred, None, pred[0].to(torch.bfloat16))
