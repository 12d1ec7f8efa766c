"""Crop decode: mae_prep_batch fed with JPEG files against the oracle's chain (decode the WHOLE
image with the oracle's decoder, then the same pipeline on the decoded pixels).  The decoder's
integer arithmetic is part of its definition, so pixels agree exactly before the resampling and
the outputs agree to the tolerance of the path."""
import numpy as np
import pytest
import torch

import oracle
import paper_2404_00509_amd as mae
from paper_2404_00509_amd import synth

from helpers import assert_close_device, check_neutral_outputs, check_prep_against_oracle, prep_to_numpy

pytestmark = pytest.mark.gpu


def _decode_all(files, offsets, sizes):
    """Oracle-decoded images in the packed layout of the decoded-input mode."""
    imgs = [oracle.jpeg_decode(files[o:o + n].tobytes()) for o, n in zip(offsets, sizes)]
    hs = np.array([i.shape[0] for i in imgs], np.int32)
    ws = np.array([i.shape[1] for i in imgs], np.int32)
    lens = hs.astype(np.int64) * ws * 3
    offs = np.zeros(len(imgs), np.int64)
    offs[1:] = np.cumsum(lens)[:-1]
    return np.concatenate([i.reshape(-1) for i in imgs]), offs, hs, ws


def _gpu_jpeg_prep(files, offsets, sizes, bf16=False, **kw):
    dev = [torch.from_numpy(a).cuda() for a in (files, offsets, sizes)]
    desc = mae.make_prep_desc(dev[0], dev[1], None, None, file_sizes=dev[2],
                              out_dtype=mae.MAE_BF16 if bf16 else mae.MAE_F32, **kw)
    buf = mae.alloc_prep_buffers(desc)
    buf.visible.fill_(float("nan"))
    buf.target.fill_(float("nan"))
    buf.crop.fill_(-7)
    mae.mae_prep_batch(desc, buf.visible, buf.mask, buf.ids_restore, buf.ids_keep, buf.target,
                       buf.crop, buf.workspace)
    torch.cuda.synchronize()
    return buf, desc


@pytest.mark.parametrize("sub", ["4:2:0", "4:4:4"])
@pytest.mark.parametrize("kind,S", [("gradient", 112), ("uniform", 64)])
def test_crop_decode_matches_full_decode(sub, kind, S):
    B = 16 if sub == "4:2:0" else 13
    files, offsets, sizes = synth.make_jpegs(kind, B, seed=60, subsampling=sub)
    L = (S // 16) ** 2
    kw = dict(out_size=S, patch=16, num_keep=oracle.num_keep(L, 0.75), seed=13, batch_index=1)
    ref = oracle.prep_batch(*_decode_all(files, offsets, sizes), **kw)
    buf, _ = _gpu_jpeg_prep(files, offsets, sizes, **kw)
    assert mae.mae_prep_status(buf.workspace) == 0
    check_prep_against_oracle(prep_to_numpy(buf), ref, what=f"{kind} {sub}")


def test_whole_image_and_tiny_crops():
    """Scale range at its ends: the crop is the whole image (every row and column of MCUs is
    decoded), or a few per cent of it (most of the file is skipped)."""
    B, S = 12, 96
    files, offsets, sizes = synth.make_jpegs("gradient", B, seed=61)
    decoded = _decode_all(files, offsets, sizes)
    L = (S // 16) ** 2
    for scale, ratio in (((1.0, 1.0), (1.0, 1.0)), ((0.02, 0.05), (0.75, 4 / 3))):
        kw = dict(out_size=S, patch=16, num_keep=L, scale=scale, ratio=ratio, seed=14,
                  batch_index=2)
        ref = oracle.prep_batch(*decoded, **kw)
        buf, _ = _gpu_jpeg_prep(files, offsets, sizes, **kw)
        check_prep_against_oracle(prep_to_numpy(buf), ref, what=f"scale {scale}")


def test_bf16_tokens_and_finetune_augmentation_from_jpeg():
    B, S = 12, 160
    files, offsets, sizes = synth.make_jpegs("gradient", B, seed=62, quality=75)
    decoded = _decode_all(files, offsets, sizes)
    L = (S // 16) ** 2
    kw = dict(out_size=S, patch=16, num_keep=L, seed=15, batch_index=0,
              aug_mode=mae.MAE_AUG_THREE_PLUS, jitter=0.3)
    ref = oracle.prep_batch(*decoded, **kw)
    buf, _ = _gpu_jpeg_prep(files, offsets, sizes, bf16=True, **kw)
    check_prep_against_oracle(prep_to_numpy(buf), ref, bf16=True, what="jpeg + 3 Aug+")


@pytest.mark.parametrize("quality,optimize", [(50, True), (98, True), (98, False)])
def test_tables_of_the_file_and_other_qualities(quality, optimize):
    """Huffman tables fitted to each image (other code lengths than the standard tables', found
    in the file) and quantisers from coarse to nearly lossless (values of up to 10 bits)."""
    B, S = 12, 96
    files, offsets, sizes = synth.make_jpegs("gradient", B, seed=64, quality=quality,
                                             optimize=optimize)
    L = (S // 16) ** 2
    kw = dict(out_size=S, patch=16, num_keep=oracle.num_keep(L, 0.75), seed=17, batch_index=4)
    ref = oracle.prep_batch(*_decode_all(files, offsets, sizes), **kw)
    buf, _ = _gpu_jpeg_prep(files, offsets, sizes, **kw)
    assert mae.mae_prep_status(buf.workspace) == 0
    check_prep_against_oracle(prep_to_numpy(buf), ref, what=f"quality {quality}")


@pytest.mark.parametrize("rows,blocks", [(0, 0), (2, 0), (0, 3), (0, 1), (3, 0)])
@pytest.mark.parametrize("sub", ["4:2:0", "4:4:4"])
def test_files_whose_rows_are_not_independent(rows, blocks, sub):
    """No restart markers at all (what an encoder writes by default), a restart interval of several
    rows of MCUs, and intervals of a few MCUs that end inside rows: the bytes decoded are the
    oracle's, so every output matches to the path's tolerance."""
    B, S = 14, 96
    kind = "uniform" if blocks == 1 else "gradient"
    files, offsets, sizes = synth.make_jpegs(kind, B, seed=66, subsampling=sub,
                                             restart_rows=rows, restart_blocks=blocks)
    decoded = _decode_all(files, offsets, sizes)
    L = (S // 16) ** 2
    for scale in ((0.2, 1.0), (1.0, 1.0), (0.02, 0.06)):
        kw = dict(out_size=S, patch=16, num_keep=oracle.num_keep(L, 0.75), scale=scale, seed=19,
                  batch_index=6)
        ref = oracle.prep_batch(*decoded, **kw)
        buf, _ = _gpu_jpeg_prep(files, offsets, sizes, **kw)
        assert mae.mae_prep_status(buf.workspace) == 0
        check_prep_against_oracle(prep_to_numpy(buf), ref,
                                  what=f"restart rows {rows} blocks {blocks} {sub} scale {scale}")


@pytest.mark.parametrize("sub", ["4:2:0", "4:4:4"])
@pytest.mark.parametrize("side", [64, 256])
def test_files_without_markers_at_the_edges_of_the_parallel_walk(sub, side):
    """Files that are one chain of codes are walked in 64 parts at once: fewer blocks than parts
    (one MCU up), flat images (thousands of blocks of a few bits), blocks longer than a part, white
    noise at quality 100 (starts that meet the chain late, or never), and a file larger than the
    memory of the parallel walk (a full-size image of noise, 4:4:4), which takes the serial one."""
    import io

    from PIL import Image
    rng = np.random.default_rng(side)
    jobs = [("flat", 24, 24, 90), ("noise", 3, 5, 100), ("noise", 16, 16, 100), ("noise", 16, 64, 100),
            ("noise", 40, 23, 75), ("flat", side, side, 90), ("ramp", side, side - 7, 95),
            ("noise", side, side, 100), ("noise", side - 1, side // 2, 60), ("ramp", side // 2, side, 30)]
    chunks = []
    for kind, h, w, quality in jobs:
        img = np.full((h, w, 3), 77, np.uint8)
        if kind == "noise":
            img = rng.integers(0, 256, (h, w, 3), dtype=np.uint8)
        elif kind == "ramp":
            img = (np.add.outer(np.arange(h) * 3, np.arange(w) * 2)[..., None]
                   + np.array([0, 40, 90])).astype(np.uint8)
        buf = io.BytesIO()
        Image.fromarray(img).save(buf, format="JPEG", quality=quality, subsampling=sub)
        chunks.append(np.frombuffer(buf.getvalue(), np.uint8))
    B = len(chunks)
    sizes = np.array([c.size for c in chunks], np.int32)
    offsets = np.zeros(B, np.int64)
    offsets[1:] = np.cumsum(sizes.astype(np.int64))[:-1]
    files = np.concatenate(chunks)
    decoded = _decode_all(files, offsets, sizes)
    S = 32
    for scale in ((1.0, 1.0), (0.1, 0.9)):
        kw = dict(out_size=S, patch=16, num_keep=2, scale=scale, seed=23, batch_index=2)
        buf, _ = _gpu_jpeg_prep(files, offsets, sizes, max_image_side=side, **kw)
        assert mae.mae_prep_status(buf.workspace) == 0
        check_prep_against_oracle(prep_to_numpy(buf), oracle.prep_batch(*decoded, **kw),
                                  what=f"{sub} side {side} scale {scale}")


def test_a_batch_that_mixes_how_its_files_are_organised():
    import io

    from PIL import Image
    B, S = 12, 112
    imgs = synth.make_images("gradient", B, seed=68)
    variants = [dict(restart_marker_rows=1), dict(), dict(restart_marker_blocks=5),
                dict(restart_marker_rows=4), dict(optimize=True), dict(restart_marker_blocks=2,
                                                                       subsampling="4:4:4")]
    chunks = []
    for b in range(B):
        buf = io.BytesIO()
        args = dict(format="JPEG", quality=85, subsampling="4:2:0")
        args.update(variants[b % len(variants)])
        Image.fromarray(synth.image_view(*imgs, b)).save(buf, **args)
        chunks.append(np.frombuffer(buf.getvalue(), np.uint8))
    sizes = np.array([c.size for c in chunks], np.int32)
    offsets = np.zeros(B, np.int64)
    offsets[1:] = np.cumsum(sizes.astype(np.int64))[:-1]
    files = np.concatenate(chunks)
    L = (S // 16) ** 2
    kw = dict(out_size=S, patch=16, num_keep=oracle.num_keep(L, 0.75), seed=21, batch_index=8)
    ref = oracle.prep_batch(*_decode_all(files, offsets, sizes), **kw)
    buf, _ = _gpu_jpeg_prep(files, offsets, sizes, **kw)
    assert mae.mae_prep_status(buf.workspace) == 0
    check_prep_against_oracle(prep_to_numpy(buf), ref, what="mixed batch")


def test_image_shapes_at_the_limits():
    """Up to 128 rows of MCUs in a file (more rows than a wavefront has lanes), a row of 63 MCUs,
    images smaller than one MCU and with ragged edges, with and without restart markers; an image
    that does not fit the side limit is flagged."""
    import io

    from PIL import Image
    shapes = [(512, 72, "4:4:4", 1), (1024, 48, "4:2:0", 1), (48, 1000, "4:2:0", 1),
              (8, 8, "4:4:4", 1), (5, 7, "4:2:0", 0), (17, 23, "4:2:0", 0), (505, 131, "4:4:4", 0),
              (1040, 64, "4:4:4", 1), (1024, 40, "4:4:4", 1), (1000, 56, "4:4:4", 0)]
    rng = np.random.default_rng(65)
    chunks = []
    for h, w, sub, rst in shapes:
        buf = io.BytesIO()
        kw = dict(restart_marker_rows=1) if rst else {}
        Image.fromarray(synth._one_image("gradient", h, w, rng)).save(
            buf, format="JPEG", quality=90, subsampling=sub, **kw)
        chunks.append(np.frombuffer(buf.getvalue(), np.uint8))
    # and the file written by hand (its own small tables, 162 bytes), after the one that is flagged
    from conftest import read_golden
    hand = next(r[1:] for r in read_golden("jpeg_hand_example.txt") if r[0] == "file")
    chunks.append(np.frombuffer(bytes.fromhex("".join(hand)), np.uint8))
    n = len(chunks)
    sizes = np.array([c.size for c in chunks], np.int32)
    offsets = np.zeros(n, np.int64)
    offsets[1:] = np.cumsum(sizes.astype(np.int64))[:-1]
    files = np.concatenate(chunks)
    S = 64
    L = (S // 16) ** 2
    keep = [b for b in range(n) if b != 7]
    # the oracle gets the hand-written image in place of the file that is too large
    stand_in = [n - 1 if b == 7 else b for b in range(n)]
    decoded = _decode_all(files, offsets[stand_in], sizes[stand_in])
    for scale in ((0.2, 1.0), (1.0, 1.0)):
        kw = dict(out_size=S, patch=16, num_keep=L, scale=scale, seed=18, batch_index=5)
        buf, _ = _gpu_jpeg_prep(files, offsets, sizes, max_image_side=1024, **kw)
        crop = buf.crop.cpu().numpy()
        assert list(np.nonzero(crop[:, 5] == 0)[0]) == [7]        # 1040 rows: beyond the limit
        ref = oracle.prep_batch(*decoded, **kw)
        sel = {k: (v[keep] if v is not None else None) for k, v in ref.items()}
        check_prep_against_oracle(prep_to_numpy(buf, rows=keep), sel, what=f"limits {scale}")


def test_the_largest_side_limit():
    """Slots of 32768 x 32768 pixels: the offsets inside one do not fit 31 bits."""
    files, offsets, sizes = synth.make_jpegs("gradient", 2, seed=75, restart_rows=0)
    kw = dict(out_size=64, patch=16, num_keep=4, seed=32, batch_index=0)
    ref = oracle.prep_batch(*_decode_all(files, offsets, sizes), **kw)
    buf, _ = _gpu_jpeg_prep(files, offsets, sizes, max_image_side=32767, **kw)
    assert mae.mae_prep_status(buf.workspace) == 0
    check_prep_against_oracle(prep_to_numpy(buf), ref, what="side limit 32767")


def test_files_the_decoder_does_not_take_are_flagged_and_take_no_part():
    import io

    from PIL import Image
    B, S = 8, 64
    imgs = synth.make_images("uniform", B, seed=63)

    def enc(b, **kw):
        buf = io.BytesIO()
        args = dict(format="JPEG", quality=90, subsampling="4:2:0", restart_marker_rows=1)
        args.update(kw)
        Image.fromarray(synth.image_view(*imgs, b)).save(buf, **args)
        return np.frombuffer(buf.getvalue(), np.uint8)

    good = [enc(b) for b in range(B)]
    gray = io.BytesIO()
    Image.fromarray(synth.image_view(*imgs, 1)).convert("L").save(gray, format="JPEG", quality=90)
    bad = {1: np.frombuffer(gray.getvalue(), np.uint8),   # one component
           3: enc(3, progressive=True),
           4: good[4][:200].copy(),                   # cut inside the tables
           6: enc(6, subsampling="4:2:2")}
    chunks = [bad.get(b, good[b]) for b in range(B)]
    # a file whose entropy-coded data is cut short: decodes (zero bits are supplied), no fault
    chunks[7] = np.concatenate([good[7][:len(good[7]) * 2 // 3], np.array([0xFF, 0xD9], np.uint8)])
    sizes = np.array([c.size for c in chunks], np.int32)
    offsets = np.zeros(B, np.int64)
    offsets[1:] = np.cumsum(sizes.astype(np.int64))[:-1]
    files = np.concatenate(chunks)
    L = (S // 16) ** 2
    kw = dict(out_size=S, patch=16, num_keep=L, seed=16, batch_index=3)
    buf, _ = _gpu_jpeg_prep(files, offsets, sizes, **kw)
    crop = buf.crop.cpu().numpy()
    flagged = sorted(int(b) for b in np.nonzero(crop[:, 5] == 0)[0])
    assert set(bad) <= set(flagged) <= set(bad) | {7}
    assert mae.mae_prep_status(buf.workspace) == len(flagged)
    # the good files give what they give on their own
    keep = [b for b in range(B) if b not in flagged]
    g_sizes = np.array([good[b].size for b in range(B)], np.int32)
    g_offsets = np.zeros(B, np.int64)
    g_offsets[1:] = np.cumsum(g_sizes.astype(np.int64))[:-1]
    ref = oracle.prep_batch(*_decode_all(np.concatenate(good), g_offsets, g_sizes), **kw)
    got = prep_to_numpy(buf, rows=keep)
    sel = {k: (v[keep] if v is not None else None) for k, v in ref.items()}
    check_prep_against_oracle(got, sel, what="good files next to bad ones")
    # flagged samples get the neutral outputs (nothing masked, identity order, zero pixels)
    for b in flagged:
        check_neutral_outputs(buf, b)


@pytest.mark.parametrize("restart_rows", [0, 1, 2])
def test_coefficients_and_planes_in_one_batch(restart_rows):
    """4:4:4 files whose crops are around half the slot: the coefficients of some fit the plane
    buffer, of the others the first rows go to the region buffer.  Tables with codes that the direct tables leave out
    (optimised, quality 100), and crops that start right of the first MCU."""
    B, S = 13, 64
    files, offsets, sizes = synth.make_jpegs("gradient", B, seed=68, quality=100, subsampling="4:4:4",
                                             restart_rows=restart_rows)
    kw = dict(out_size=S, patch=16, num_keep=4, scale=(0.35, 0.75), seed=24, batch_index=1)
    ref = oracle.prep_batch(*_decode_all(files, offsets, sizes), **kw)
    buf, _ = _gpu_jpeg_prep(files, offsets, sizes, **kw)
    assert mae.mae_prep_status(buf.workspace) == 0
    check_prep_against_oracle(prep_to_numpy(buf), ref, what=f"restart rows {restart_rows}")


@pytest.mark.parametrize("restart_rows", [0, 1])
@pytest.mark.parametrize("side,shapes", [
    (64, [(64, 64), (57, 64), (64, 49), (33, 64), (40, 60), (64, 8)]),
    (256, [(256, 256), (250, 256), (256, 130), (129, 256), (180, 200), (256, 64)]),
    # rows of more than 64 MCUs are transformed in several steps; the whole slot goes by planes
    (576, [(576, 576), (568, 576), (576, 565), (300, 576), (576, 520)])])
def test_coefficients_of_up_to_twice_the_plane_slot(side, shapes, restart_rows):
    """Whole 4:4:4 images, from the whole slot down to crops that the plane buffer holds alone."""
    import io

    from PIL import Image
    rng = np.random.default_rng(side)
    chunks = []
    for h, w in shapes:
        buf = io.BytesIO()
        kw = dict(restart_marker_rows=1) if restart_rows else {}
        Image.fromarray(synth._one_image("gradient", h, w, rng)).save(
            buf, format="JPEG", quality=90, subsampling="4:4:4", **kw)
        chunks.append(np.frombuffer(buf.getvalue(), np.uint8))
    files, offsets, sizes = _join(chunks)
    decoded = _decode_all(files, offsets, sizes)
    for scale, ratio in (((1.0, 1.0), (0.61, 1.6)), ((0.4, 0.9), (0.75, 4 / 3))):
        kw = dict(out_size=96, patch=16, num_keep=9, scale=scale, ratio=ratio, seed=33,
                  batch_index=3)
        ref = oracle.prep_batch(*decoded, **kw)
        buf, _ = _gpu_jpeg_prep(files, offsets, sizes, max_image_side=side, **kw)
        assert mae.mae_prep_status(buf.workspace) == 0
        check_prep_against_oracle(prep_to_numpy(buf), ref, what=f"side {side} scale {scale}")


@pytest.mark.parametrize("restart_rows", [0, 1])
def test_large_files_with_wrong_bytes_next_to_good_ones(restart_rows):
    """Noise in the entropy-coded data of 4:4:4 files whose rows spill: wrong pixels or a flagged
    sample; the files around them in the buffers are what they are alone."""
    B, S = 7, 64
    files, offsets, sizes = synth.make_jpegs("gradient", B, seed=77, quality=95, subsampling="4:4:4",
                                             restart_rows=restart_rows)
    decoded = _decode_all(files, offsets, sizes)
    files = files.copy()
    rng = np.random.default_rng(78)
    wrong = (1, 2, 5)
    for b in wrong:
        lo, hi = offsets[b] + sizes[b] // 3, offsets[b] + sizes[b] - 200
        files[lo:hi] = rng.integers(0, 255, hi - lo)        # no 0xFF: no marker among them
    kw = dict(out_size=S, patch=16, num_keep=4, scale=(1.0, 1.0), ratio=(0.61, 1.6), seed=35,
              batch_index=1)
    ref = oracle.prep_batch(*decoded, **kw)
    buf, _ = _gpu_jpeg_prep(files, offsets, sizes, **kw)
    assert bool(torch.isfinite(buf.target).all()) and bool(torch.isfinite(buf.visible).all())
    keep = [b for b in range(B) if b not in wrong]
    sel = {k: (v[keep] if v is not None else None) for k, v in ref.items()}
    check_prep_against_oracle(prep_to_numpy(buf, rows=keep), sel, what="good files")


def test_files_without_markers_whose_data_ends_early():
    """Inside the last row (zero bits follow: rows are then not decoded in pieces), or rows before it
    (no marker ends the data: the rows behind it are zero bits, too)."""
    one, _, lens = synth.make_jpegs("gradient", 1, seed=69, restart_rows=0)
    cuts = [0, 2, 9, 60, 400, lens[0] // 2]
    chunks = [one[:lens[0] - c] for c in cuts]
    sizes = np.array([c.size for c in chunks], np.int32)
    offsets = np.zeros(len(cuts), np.int64)
    offsets[1:] = np.cumsum(sizes.astype(np.int64))[:-1]
    files = np.concatenate(chunks)
    kw = dict(out_size=96, patch=16, num_keep=9, scale=(1.0, 1.0), ratio=(1.0, 1.0), seed=25)
    ref = oracle.prep_batch(*_decode_all(files, offsets, sizes), **kw)
    buf, _ = _gpu_jpeg_prep(files, offsets, sizes, **kw)
    crop = buf.crop.cpu().numpy()
    assert list(crop[:, 5]) == [1, 1, 1, 1, 1, 1]
    check_prep_against_oracle(prep_to_numpy(buf), ref, what="cut files")


def test_files_of_maximum_side_500():
    """The size of the paper's crop-decode benchmark: 24 to 32 rows of MCUs per image."""
    B, S = 6, 224
    files, offsets, sizes = synth.make_jpegs("gradient500", B, seed=67)
    L = (S // 16) ** 2
    kw = dict(out_size=S, patch=16, num_keep=oracle.num_keep(L, 0.75), seed=20, batch_index=7)
    ref = oracle.prep_batch(*_decode_all(files, offsets, sizes), **kw)
    buf, _ = _gpu_jpeg_prep(files, offsets, sizes, max_image_side=512, **kw)
    assert mae.mae_prep_status(buf.workspace) == 0
    check_prep_against_oracle(prep_to_numpy(buf), ref, what="side 500")


@pytest.mark.parametrize("B,side", [(1025, 256), (2051, 256), (1027, 512)])
def test_batches_whose_wavefronts_share_images(B, side):
    """The entropy kernel takes one, two or four images per wavefront by the batch's size (two at most
    beyond 256 pixels): batches just over the lines, with the last group partly filled, whose groups
    mix files in every organisation (rows, chains whose rows are taken in pieces, 4:4:4 crops that
    spill, up to 128 rows per group, intervals that end inside rows) with files that are refused."""
    import io

    from PIL import Image
    kind = "gradient" if side == 256 else "gradient500"
    n = 22                                   # no multiple of four: every group is another mixture
    imgs = synth.make_images(kind, n, seed=76)
    variants = [dict(restart_marker_rows=1), dict(), dict(subsampling="4:4:4", restart_marker_rows=1),
                dict(subsampling="4:4:4"), dict(progressive=True), dict(restart_marker_blocks=5),
                dict(subsampling="4:4:4", restart_marker_rows=1, narrow=True), dict(optimize=True)]
    chunks, refused = [], []
    for i in range(n):
        args = dict(format="JPEG", quality=85, subsampling="4:2:0")
        args.update(variants[i % len(variants)])
        view = synth.image_view(*imgs, i)
        if args.pop("narrow", False):
            view = np.ascontiguousarray(view[:, :100])
        refused.append("progressive" in args)
        buf = io.BytesIO()
        Image.fromarray(view).save(buf, **args)
        chunks.append(np.frombuffer(buf.getvalue(), np.uint8))
    files, first, lens = _join(chunks)
    pick = np.arange(B) % n
    # (the oracle gets the first file's image in place of a refused one)
    stand_in = np.where(refused, 0, np.arange(n))
    images, offs, hs, ws = _decode_all(files, first[stand_in], lens[stand_in])
    ref = dict(out_size=32, patch=16, num_keep=2, scale=(0.2, 1.0), seed=34, batch_index=4)
    buf, _ = _gpu_jpeg_prep(files, first[pick], lens[pick], max_image_side=side, **ref)
    ref = oracle.prep_batch(images, offs[pick], hs[pick], ws[pick], **ref)
    bad = np.array(refused)[pick]
    np.testing.assert_array_equal(buf.crop[:, 5].cpu().numpy(), np.where(bad, 0, 1))
    keep = np.nonzero(~bad)[0]
    sel = {k: (v[keep] if v is not None else None) for k, v in ref.items()}
    check_prep_against_oracle(prep_to_numpy(buf, rows=keep), sel, what=f"{B} files, side {side}")
    for b in np.nonzero(bad)[0][[0, -1]]:
        check_neutral_outputs(buf, int(b))


def test_jpeg_input_on_a_side_stream_and_in_a_captured_graph():
    """The JPEG path enqueues kernels only (header, crop draws, tables, decode, colour, resample,
    augmentation): it can run on any stream and be captured; every replay is checked."""
    B, S = 8, 96
    files, offsets, sizes = synth.make_jpegs("gradient", B, seed=66)
    L = (S // 16) ** 2
    kw = dict(out_size=S, patch=16, num_keep=L, seed=19, batch_index=6,
              aug_mode=mae.MAE_AUG_THREE_PLUS, jitter=0.3)
    ref = oracle.prep_batch(*_decode_all(files, offsets, sizes), **kw)
    dev = [torch.from_numpy(a).cuda() for a in (files, offsets, sizes)]
    desc = mae.make_prep_desc(dev[0], dev[1], None, None, file_sizes=dev[2], **kw)
    buf = mae.alloc_prep_buffers(desc)

    def step(stream):
        mae.mae_prep_batch(desc, buf.visible, buf.mask, buf.ids_restore, buf.ids_keep, buf.target,
                           buf.crop, buf.workspace, stream=stream)

    def wipe():
        buf.visible.fill_(float("nan"))
        buf.target.fill_(float("nan"))
        buf.ids_restore.fill_(-1)
        buf.workspace.zero_()
        torch.cuda.synchronize()

    side = torch.cuda.Stream()
    wipe()
    with torch.cuda.stream(side):
        step(side)
    side.synchronize()
    check_prep_against_oracle(prep_to_numpy(buf), ref, what="side stream")
    graph = torch.cuda.CUDAGraph()
    wipe()
    with torch.cuda.graph(graph):
        step(torch.cuda.current_stream())
    for replay in range(3):
        wipe()
        graph.replay()
        torch.cuda.synchronize()
        check_prep_against_oracle(prep_to_numpy(buf), ref, what=f"graph replay {replay}")
        buf.target.mul_(1.0)          # eager work between replays
        torch.cuda.synchronize()


def test_crop_decode_full_size_every_image():
    """The bench's launch: 4096 files (max side 256, quality 90, 4:2:0) -> 224 px, every image
    against the oracle's path on the oracle-decoded images."""
    from concurrent.futures import ThreadPoolExecutor

    wl = synth.WORKLOADS["c4"]
    files, offsets, sizes = synth.make_jpegs(wl.kind, wl.B, seed=0)
    K = oracle.num_keep(wl.L, wl.mask_ratio)
    kw = dict(out_size=wl.out_size, patch=wl.patch, num_keep=K, seed=5, batch_index=9)
    buf, _ = _gpu_jpeg_prep(files, offsets, sizes, **kw)
    assert mae.mae_prep_status(buf.workspace) == 0
    # whole-file decode by the oracle (the C call releases the interpreter lock)
    blobs = [files[o:o + n].tobytes() for o, n in zip(offsets, sizes)]
    with ThreadPoolExecutor(16) as pool:
        imgs = list(pool.map(oracle.jpeg_decode, blobs))
    lens = np.array([im.size for im in imgs], np.int64)
    offs = np.zeros(wl.B, np.int64)
    offs[1:] = np.cumsum(lens)[:-1]
    decoded = (np.concatenate([im.reshape(-1) for im in imgs]), offs,
               np.array([im.shape[0] for im in imgs], np.int32),
               np.array([im.shape[1] for im in imgs], np.int32))
    for lo in range(0, wl.B, 256):
        hi = min(lo + 256, wl.B)
        ref = oracle.prep_batch(*decoded, b_begin=lo, b_end=hi, **kw)
        what = f"files {lo}..{hi}"
        for k in ("ids_restore", "ids_keep", "mask"):
            np.testing.assert_array_equal(getattr(buf, k)[lo:hi].cpu().numpy(), ref[k],
                                          err_msg=what + k)
        np.testing.assert_array_equal(buf.crop[lo:hi, :5].cpu().numpy(), ref["crop"], err_msg=what)
        assert_close_device(buf.target[lo:hi], ref["target"], what=what + " target")
        assert_close_device(buf.visible[lo:hi], ref["visible"], what=what + " visible")


# ---- the files' row index ------------------------------------------------------------------------
def _row_index(files, offsets, sizes, max_image_side=0):
    """mae_jpeg_index over the files: (index tensor [B, bytes per file], device inputs)."""
    dev = [torch.from_numpy(a).cuda() for a in (files, offsets, sizes)]
    desc = mae.make_prep_desc(dev[0], dev[1], None, None, file_sizes=dev[2], out_size=32, patch=16,
                              num_keep=1, max_image_side=max_image_side)
    index = torch.full((mae.mae_jpeg_index_bytes(desc),), 0xEE, dtype=torch.uint8, device="cuda")
    ws = torch.empty(mae.mae_prep_workspace_bytes(desc), dtype=torch.uint8, device="cuda")
    mae.mae_jpeg_index(desc, index, ws)
    torch.cuda.synchronize()
    return index.view(len(sizes), -1), dev


def _prep_with_index(dev, index, **kw):
    desc = mae.make_prep_desc(dev[0], dev[1], None, None, file_sizes=dev[2], row_index=index, **kw)
    buf = mae.alloc_prep_buffers(desc)
    buf.visible.fill_(float("nan"))
    buf.target.fill_(float("nan"))
    buf.crop.fill_(-7)
    mae.mae_prep_batch(desc, buf.visible, buf.mask, buf.ids_restore, buf.ids_keep, buf.target,
                       buf.crop, buf.workspace)
    torch.cuda.synchronize()
    return buf


@pytest.mark.parametrize("sub", ["4:2:0", "4:4:4"])
def test_row_index_replaces_the_walk_through_the_file(sub):
    """The index of a file (computed once, whatever crops come later) gives the decoder the same
    row starts as walking through the file does: same outputs bit for bit, for files without
    restart markers, with odd intervals and with a marker per row, mixed in one batch, for
    several batches of crops, and for a batch gathered from the indexed files in another order."""
    B, S = 15, 96
    parts = [synth.make_jpegs("gradient", B, seed=70, subsampling=sub, restart_rows=r,
                              restart_blocks=k) for r, k in ((0, 0), (1, 0), (0, 3))]
    pick = np.arange(B) % 3  # file b comes from organisation b mod 3
    blobs = [parts[pick[b]][0][parts[pick[b]][1][b]:parts[pick[b]][1][b] + parts[pick[b]][2][b]]
             for b in range(B)]
    sizes = np.array([len(x) for x in blobs], np.int32)
    offsets = np.zeros(B, np.int64)
    offsets[1:] = np.cumsum((sizes.astype(np.int64) + 7) // 8 * 8)[:-1]
    files = np.zeros(int(offsets[-1] + (sizes[-1] + 7) // 8 * 8), np.uint8)
    for b in range(B):
        files[offsets[b]:offsets[b] + sizes[b]] = blobs[b]
    decoded = _decode_all(files, offsets, sizes)
    index, dev = _row_index(files, offsets, sizes)
    L = (S // 16) ** 2
    for batch_index, scale in ((0, (0.2, 1.0)), (1, (1.0, 1.0)), (2, (0.03, 0.1))):
        kw = dict(out_size=S, patch=16, num_keep=oracle.num_keep(L, 0.75), scale=scale, seed=23,
                  batch_index=batch_index)
        ref = oracle.prep_batch(*decoded, **kw)
        plain, _ = _gpu_jpeg_prep(files, offsets, sizes, **kw)
        got = _prep_with_index(dev, index, **kw)
        assert mae.mae_prep_status(got.workspace) == 0
        check_prep_against_oracle(prep_to_numpy(got), ref, what=f"index, batch {batch_index}")
        assert torch.equal(got.target, plain.target) and torch.equal(got.visible, plain.visible)
    # another batch of the same files: reversed order, index entries gathered like the files
    order = np.arange(B)[::-1].copy()
    sizes2 = sizes[order]
    offsets2 = np.zeros(B, np.int64)
    offsets2[1:] = np.cumsum((sizes2.astype(np.int64) + 7) // 8 * 8)[:-1]
    files2 = np.zeros(int(offsets2[-1] + (sizes2[-1] + 7) // 8 * 8), np.uint8)
    for i, b in enumerate(order):
        files2[offsets2[i]:offsets2[i] + sizes2[i]] = blobs[b]
    dev2 = [torch.from_numpy(a).cuda() for a in (files2, offsets2, sizes2)]
    index2 = index[torch.from_numpy(order).cuda()].contiguous()
    kw = dict(out_size=S, patch=16, num_keep=L, seed=24, batch_index=5)
    ref = oracle.prep_batch(*_decode_all(files2, offsets2, sizes2), **kw)
    got = _prep_with_index(dev2, index2, **kw)
    assert mae.mae_prep_status(got.workspace) == 0
    check_prep_against_oracle(prep_to_numpy(got), ref, what="gathered index")


def test_row_index_entries_are_checked_before_use():
    """The index is the caller's memory.  Entries that cannot belong to their file (zeros, noise,
    the entries of another file) give samples flagged invalid or wrong pixels; the call returns,
    every output is written, and good entries next to them still decode exactly."""
    B, S = 12, 64
    files, offsets, sizes = synth.make_jpegs("gradient", B, seed=71, restart_rows=0)
    decoded = _decode_all(files, offsets, sizes)
    index, dev = _row_index(files, offsets, sizes)
    bad = index.clone()
    bad[1].zero_()                                       # position 0: before the scan data
    rng = np.random.default_rng(5)
    bad[4] = torch.from_numpy(rng.integers(0, 256, bad.shape[1], dtype=np.uint8)).cuda()
    bad[7] = index[8]                                    # another file's row starts
    bad[10].fill_(0xFF)                                  # negative position and bit count
    L = (S // 16) ** 2
    kw = dict(out_size=S, patch=16, num_keep=L, seed=25, batch_index=0)
    ref = oracle.prep_batch(*decoded, **kw)
    got = _prep_with_index(dev, bad.contiguous(), **kw)
    n_bad = mae.mae_prep_status(got.workspace)
    assert 3 <= n_bad <= 4            # only another file's entries may decode (to wrong pixels)
    out = prep_to_numpy(got)
    assert np.isfinite(out["target"]).all() and np.isfinite(out["visible"]).all()
    good = np.array([b for b in range(B) if b not in (1, 4, 7, 10)])
    assert np.all(out["crop"][good, 5] == 1)
    np.testing.assert_array_equal(out["ids_restore"][good], ref["ids_restore"][good])
    assert_close_device(got.target[torch.from_numpy(good).cuda()], ref["target"][good],
                        what="good entries")
    for b in (1, 4, 10):
        check_neutral_outputs(got, b)


def test_row_index_of_files_the_decoder_does_not_take():
    """A file that is not decodable gets an index of unknown rows, and so does every row a file
    does not have; with such an index the sample is flagged exactly as without one."""
    B = 6
    files, offsets, sizes = synth.make_jpegs("gradient", B, seed=72, restart_rows=0)
    files = files.copy()
    files[offsets[2] + 2:offsets[2] + 40] = 0            # the header of file 2 destroyed
    index, dev = _row_index(files, offsets, sizes)
    rows = index.view(B, -1, 32)
    pos = rows[:, :, :4].contiguous().view(torch.int32).view(B, -1).cpu().numpy()
    assert np.all(pos[2] == -1)
    for b in (0, 1, 3, 4, 5):
        h = oracle.jpeg_decode(files[offsets[b]:offsets[b] + sizes[b]].tobytes()).shape[0]
        n_rows = (h + 15) // 16
        assert np.all(pos[b, :n_rows] > 0) and np.all(pos[b, n_rows:] == -1)
        assert np.all(np.diff(pos[b, :n_rows]) > 0)      # rows follow each other in the file
    kw = dict(out_size=64, patch=16, num_keep=4, seed=26, batch_index=0)
    got = _prep_with_index(dev, index, **kw)
    assert mae.mae_prep_status(got.workspace) == 1
    assert prep_to_numpy(got)["crop"][2, 5] == 0


def test_row_index_with_large_files_augmentation_and_the_loss_without_target():
    """The index under the other modes of the call: files of maximum side 500 (64 index rows per
    file), the finetuning augmentation, and the loss that reads the decoded regions again."""
    B, S = 6, 128
    files, offsets, sizes = synth.make_jpegs("gradient500", B, seed=73, restart_rows=0)
    decoded = _decode_all(files, offsets, sizes)
    index, dev = _row_index(files, offsets, sizes, max_image_side=512)
    assert index.shape[1] == 64 * 32
    L = (S // 16) ** 2
    kw = dict(out_size=S, patch=16, num_keep=L, seed=27, batch_index=1, max_image_side=512,
              aug_mode=mae.MAE_AUG_THREE_PLUS, jitter=0.3)
    ref = oracle.prep_batch(*decoded, **{k: v for k, v in kw.items() if k != "max_image_side"})
    got = _prep_with_index(dev, index, **kw)
    assert mae.mae_prep_status(got.workspace) == 0
    check_prep_against_oracle(prep_to_numpy(got), ref, what="index, side 500, 3 Aug+")

    # pretraining step without a stored target on the same files
    K = oracle.num_keep(L, 0.75)
    kw = dict(out_size=S, patch=16, num_keep=K, seed=28, batch_index=2, max_image_side=512)
    ref = oracle.prep_batch(*decoded, **{k: v for k, v in kw.items() if k != "max_image_side"})
    desc = mae.make_prep_desc(dev[0], dev[1], None, None, file_sizes=dev[2], row_index=index, **kw)
    buf = mae.alloc_prep_buffers(desc, want_target=False)
    mae.mae_prep_batch(desc, buf.visible, buf.mask, buf.ids_restore, buf.ids_keep, None, buf.crop,
                       buf.workspace)
    M = B * (L - K)
    pred_host = synth.make_pred(9, B, L, 768)
    pred = torch.from_numpy(pred_host).cuda()
    ldesc = mae.make_loss_desc(pred, None, buf.mask, num_masked=M)
    lws = torch.empty(mae.mae_loss_from_images_workspace_bytes(desc, ldesc), dtype=torch.uint8,
                      device="cuda")
    loss = torch.zeros(1, device="cuda")
    grad = torch.empty_like(pred)
    mae.mae_normpix_loss_from_images(desc, buf.workspace, ldesc, loss, grad, lws)
    torch.cuda.synchronize()
    ref_loss, ref_grad, _ = oracle.normpix_loss(pred_host, ref["target"], ref["mask"], num_masked=M)
    assert abs(loss.item() - ref_loss) <= 1e-5 + 1e-5 * abs(ref_loss)
    from helpers import check_grad
    check_grad(grad.cpu().numpy(), ref_grad, 768, M, what="index + loss from images")


def _join(chunks):
    """Files back to back: (bytes, offsets, sizes)."""
    sizes = np.array([c.size for c in chunks], np.int32)
    offsets = np.zeros(len(chunks), np.int64)
    offsets[1:] = np.cumsum(sizes.astype(np.int64))[:-1]
    return np.concatenate(chunks), offsets, sizes


def _flat(h, w, value, sub, **kw):
    import io

    from PIL import Image
    buf = io.BytesIO()
    Image.fromarray(np.full((h, w, 3), value, np.uint8)).save(buf, format="JPEG", quality=90,
                                                             subsampling=sub, **kw)
    return np.frombuffer(buf.getvalue(), np.uint8)


@pytest.mark.parametrize("indexed", [False, True])
@pytest.mark.parametrize("side", [64, 256])
def test_last_rows_of_a_few_bits(side, indexed):
    """A flat row of MCUs is as short as 14 bits (one MCU, 4:4:4, the standard's tables) or less
    (tables fitted to the file): complete files whose last rows hold fewer bits than the decoder's
    bit buffer, walked in parallel (no markers), serially (an interval of several rows, in which
    the last row but one of an interval is as short), and through the index."""
    shapes = [(24, 8, "4:4:4", {}), (16, 8, "4:4:4", dict(optimize=True)),
              (32, 32, "4:2:0", dict(optimize=True)), (48, 16, "4:2:0", {}),
              (40, 16, "4:4:4", dict(optimize=True)), (64, 40, "4:2:0", {})]
    chunks = [_flat(h, w, value, sub, **kw, **rst) for h, w, sub, kw in shapes
              for value in (0, 77, 255) for rst in ({}, dict(restart_marker_rows=2))]
    files, offsets, sizes = _join(chunks)
    decoded = _decode_all(files, offsets, sizes)
    for lo, scale in ((0.61, (1.0, 1.0)), (0.75, (0.2, 1.0))):
        kw = dict(out_size=32, patch=16, num_keep=2, scale=scale, ratio=(lo, 1 / lo), seed=31,
                  batch_index=2)
        ref = oracle.prep_batch(*decoded, **kw)
        if indexed:
            index, dev = _row_index(files, offsets, sizes, max_image_side=side)
            buf = _prep_with_index(dev, index, max_image_side=side, **kw)
        else:
            buf, _ = _gpu_jpeg_prep(files, offsets, sizes, max_image_side=side, **kw)
        assert mae.mae_prep_status(buf.workspace) == 0
        check_prep_against_oracle(prep_to_numpy(buf), ref, what=f"short rows, scale {scale}")


@pytest.mark.parametrize("indexed", [False, True])
@pytest.mark.parametrize("sub", ["4:2:0", "4:4:4"])
def test_files_cut_short_with_and_without_an_end_marker(sub, indexed):
    """A file that simply stops is decoded with zero bits from there on, as the oracle does, wherever
    it stops; a file whose data a marker ends before the crop's last row is flagged."""
    one, _, lens = synth.make_jpegs("gradient", 1, seed=69, restart_rows=0, subsampling=sub)
    n = int(lens[0])
    cuts = [n // 2, n // 3, 3 * n // 4, 2000, 1]
    chunks = [one[:n - c] for c in cuts]
    eoi = np.array([0xFF, 0xD9], np.uint8)
    chunks += [np.concatenate([one[:n - c], eoi]) for c in cuts[:3]]
    files, offsets, sizes = _join(chunks)
    kw = dict(out_size=96, patch=16, num_keep=9, scale=(1.0, 1.0), ratio=(1.0, 1.0), seed=25)
    ref = oracle.prep_batch(*_decode_all(files, offsets, sizes), **kw)
    if indexed:
        index, dev = _row_index(files, offsets, sizes)
        buf = _prep_with_index(dev, index, **kw)
    else:
        buf, _ = _gpu_jpeg_prep(files, offsets, sizes, **kw)
    assert buf.crop[:, 5].tolist() == [1] * len(cuts) + [0] * 3
    keep = list(range(len(cuts)))
    sel = {k: (v[keep] if v is not None else None) for k, v in ref.items()}
    check_prep_against_oracle(prep_to_numpy(buf, rows=keep), sel, what="cut files")
    for b in range(len(cuts), len(chunks)):
        check_neutral_outputs(buf, b)


def _rewrite_scan(file, rng, restart_rows):
    """The file (4:4:4, sides multiples of 8) with entropy-coded data that is mostly ones: every block a
    random DC difference, up to three coefficients 1023 behind runs of 15 zeros (26 bits, 25 of them
    ones, next to each other), end of block."""
    d = file.tobytes()
    codes, pos = {}, 2
    while True:
        m, n = d[pos + 1], int.from_bytes(d[pos + 2:pos + 4], "big")
        if m == 0xC0:
            rows, cols = (int.from_bytes(d[pos + 5 + 2 * i:pos + 7 + 2 * i], "big") // 8 for i in (0, 1))
        o = pos + 4
        while m == 0xC4 and o < pos + 2 + n:
            code, sym = 0, o + 17
            for length in range(1, 17):
                for _ in range(d[o + length]):
                    codes[d[o], d[sym]] = format(code, f"0{length}b")
                    code, sym = code + 1, sym + 1
                code <<= 1
            o = sym
        pos += 2 + n
        if m == 0xDA:
            break
    out, bits = bytearray(d[:pos]), ""

    def flush():
        nonlocal bits
        bits += "1" * (-len(bits) % 8)
        out.extend(bytes(int(bits[i:i + 8], 2) for i in range(0, len(bits), 8)).replace(b"\xff", b"\xff\0"))
        bits = ""
    for row in range(rows):
        for _ in range(cols):
            for t in (0, 1, 1):
                size = int(rng.integers(0, 5))
                bits += codes[t, size] + "".join(rng.choice(["0", "1"], size))
                bits += (codes[16 + t, 0xFA] + "1" * 10) * int(rng.integers(0, 4)) + codes[16 + t, 0]
        if restart_rows and row + 1 < rows:
            flush()
            out.extend((0xFF, 0xD0 + row % 8))
    flush()
    return np.frombuffer(bytes(out) + b"\xff\xd9", np.uint8)


@pytest.mark.parametrize("restart_rows", [0, 1])
def test_stuffed_bytes_at_all_places_of_a_dword(restart_rows):
    """Byte stuffing is taken out four bytes at a time, byte by byte where more than one of them goes:
    0xFF at every place of a dword, next to each other too, and in front of the restart markers.  The
    rows' states come from the markers or the walk, and from an index."""
    rng = np.random.default_rng(90)
    kw = {"restart_marker_rows": 1} if restart_rows else {}
    files, offsets, sizes = _join([_rewrite_scan(_flat(64 + 8 * i, 72, 100, "4:4:4", **kw), rng, restart_rows)
                                   for i in range(11)])
    stuffed = np.flatnonzero((files[:-1] == 0xFF) & (files[1:] == 0))
    pairs = np.intersect1d(stuffed, stuffed + 2)     # FF 00 FF 00
    for at in (stuffed, pairs):
        assert np.bincount(at % 4, minlength=4).min() > 500
    kw = dict(out_size=64, patch=16, num_keep=4, seed=27, batch_index=4)
    ref = oracle.prep_batch(*_decode_all(files, offsets, sizes), **kw)
    buf, _ = _gpu_jpeg_prep(files, offsets, sizes, **kw)
    assert mae.mae_prep_status(buf.workspace) == 0
    check_prep_against_oracle(prep_to_numpy(buf), ref, what=f"stuffed bytes, restart {restart_rows}")
    index, dev = _row_index(files, offsets, sizes)
    got = _prep_with_index(dev, index, **kw)
    assert torch.equal(got.target, buf.target) and torch.equal(got.visible, buf.visible)


@pytest.mark.parametrize("B,side", [(23, 512), (513, 512), (1025, 512)])
def test_the_parallel_walk_by_several_wavefronts(B, side):
    """Files without markers are walked by four wavefronts in batches of up to 512, by two up to 1024
    and by one beyond, with 64 to 256 parts by the length of the data: just over a wavefront's parts,
    parts that end in the last wavefront, all of them taken; flat images and single MCUs next to them,
    noise, data that simply stops and data that a marker ends too early."""
    import io

    from PIL import Image
    rng = np.random.default_rng(side)
    jobs = [("noise", 0.26, 100), ("noise", 0.31, 90), ("ramp", 1.0, 95), ("noise", 0.5, 100), ("flat", 1.0, 90),
            ("noise", 0.9, 75), ("noise", 0.05, 90), ("noise", 1.0, 60), ("noise", 0.5, 75)]
    chunks = []
    for kind, part, quality in jobs:
        h = w = max(8, int(part * side) - 3)
        img = np.full((h, w, 3), 77, np.uint8)
        if kind == "noise":
            img = rng.integers(0, 256, (h, w, 3), dtype=np.uint8)
        elif kind == "ramp":
            img = (np.add.outer(np.arange(h) * 3, np.arange(w) * 2)[..., None]
                   + np.array([0, 40, 90])).astype(np.uint8)
        buf = io.BytesIO()
        Image.fromarray(img).save(buf, format="JPEG", quality=quality, subsampling="4:2:0")
        chunks.append(np.frombuffer(buf.getvalue(), np.uint8))
    bits = np.array([8 * c.size for c in chunks])
    assert bits.min() < 64 * 2304 and bits.max() > 256 * 2304
    assert ((bits > 66 * 2304) & (bits < 128 * 2304)).any() and ((bits > 130 * 2304) & (bits < 250 * 2304)).any()
    n = len(chunks)
    for i in (3, 7):  # stops; ends with a marker
        chunks.append(chunks[i][:chunks[i].size * 2 // 3])
    chunks.append(np.concatenate([chunks[7][:chunks[7].size // 2], np.array([0xFF, 0xD9], np.uint8)]))
    files, first, lens = _join(chunks)
    pick = np.arange(B) % len(chunks)
    images, offs, hs, ws = _decode_all(files, first, lens)
    kw = dict(out_size=32, patch=16, num_keep=2, scale=(1.0, 1.0), ratio=(1.0, 1.0), seed=35, batch_index=1)
    buf, _ = _gpu_jpeg_prep(files, first[pick], lens[pick], max_image_side=side, **kw)
    ref = oracle.prep_batch(images, offs[pick], hs[pick], ws[pick], **kw)
    keep = np.flatnonzero(pick != n + 2)
    np.testing.assert_array_equal(buf.crop[:, 5].cpu().numpy(), pick != n + 2)
    sel = {k: (v[keep] if v is not None else None) for k, v in ref.items()}
    check_prep_against_oracle(prep_to_numpy(buf, rows=keep), sel, what=f"{B} files, side {side}")
    if B < 64:  # the index comes from the same walk, over whole images
        index, dev = _row_index(files, first[pick], lens[pick], max_image_side=side)
        got = _prep_with_index(dev, index, max_image_side=side, **kw)
        keep = torch.from_numpy(keep).cuda()
        assert torch.equal(got.target[keep], buf.target[keep])
