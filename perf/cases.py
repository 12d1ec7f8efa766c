"""What the library's users run, as measurable cases through its public entry points.

A case is one of four operations, with the sizes of a real call:

  step     one pretraining batch: mae_prep_batch and, with it, the reconstruction loss and its
           gradient ("loss": "stored" = mae_normpix_loss on the stored target, "images" =
           mae_normpix_loss_from_images, "none" = the input pipeline alone, as an evaluation or a
           loader uses it)
  embed    the encoder's patch embedding of the visible tokens
  augment  one finetuning batch: mae_prep_batch with "3 Aug" / "3 Aug+", every patch kept
  jpeg     one pretraining batch read from JPEG files (crop decode)

Every pass builds its descriptors, as a training loop does for each new batch; buffers and
workspaces are allocated once, as such a loop also does.
"""
from __future__ import annotations

from concurrent.futures import ThreadPoolExecutor

import numpy as np
import torch

import paper_2404_00509_amd as mae
from paper_2404_00509_amd import synth

KINDS = {128: "uniform", 256: "gradient", 500: "gradient500"}  # by the images' largest side
MEAN_PIXELS = {128: 96 * 96, 256: 256 * 208, 500: 500 * 406}   # of such an image


def _step(name, B, side, out, patch, ratio, bf16, loss):
    return {"name": name, "op": "step", "B": B, "side": side, "out": out, "patch": patch,
            "ratio": ratio, "bf16": bf16, "loss": loss}


def listed():
    return [
        # a smoke-sized batch of small images (a quick run, a unit of a sweep): launches and latency
        _step("step_112_b64", 64, 128, 112, 16, 0.75, False, "stored"),
        # the 192-pixel stage of progressive pretraining at a per-GPU batch of 1024
        _step("step_192_b1024", 1024, 256, 192, 16, 0.75, False, "stored"),
        # the headline pretraining batch: 224 pixels, ViT-B/16, 4096 images
        _step("step_224_b4096", 4096, 256, 224, 16, 0.75, False, "stored"),
        # the same at patch 14 with bf16 tokens and predictions (ViT-L/14-style inputs)
        _step("step_224_p14_bf16_b4096", 4096, 256, 224, 14, 0.75, True, "stored"),
        # the headline batch without a stored target (the loss takes the pixels from the images)
        _step("step_224_images_b4096", 4096, 256, 224, 16, 0.75, False, "images"),
        # odd sizes: the last, ragged batch of an epoch, an odd patch size, 80 % masked
        _step("step_225_p15_b333", 333, 256, 225, 15, 0.80, False, "stored"),
        # patch embedding of the headline batch's visible tokens, ViT-B width
        {"name": "embed_768_b4096", "op": "embed", "B": 4096, "K": 49, "L": 196, "D": 768,
         "E": 768, "f32_out": False},
        # patch 14 at ViT-L width and a batch of 512: D is no multiple of the matrix tile
        {"name": "embed_588_1024_b512", "op": "embed", "B": 512, "K": 64, "L": 256, "D": 588,
         "E": 1024, "f32_out": False},
        # finetuning, first stage of the progressive schedule (160 pixels, "3 Aug")
        {"name": "augment_160_b1024", "op": "augment", "B": 1024, "side": 256, "stage": 1,
         "plus": False, "patch": 16, "bf16": False},
        # finetuning, last stage (224 pixels, "3 Aug+" with colour jitter), full batch
        {"name": "augment_224_plus_b4096", "op": "augment", "B": 4096, "side": 256, "stage": 3,
         "plus": True, "patch": 16, "bf16": False},
        # pretraining from JPEG files of a dataset written for the loader (restart marker per row)
        {"name": "jpeg_rows_224_b4096", "op": "jpeg", "B": 4096, "side": 256, "out": 224,
         "patch": 16, "ratio": 0.75, "bf16": False, "files": "rows"},
        # ... from JPEG files as an encoder writes them by default, read for the first time
        {"name": "jpeg_plain_224_b1024", "op": "jpeg", "B": 1024, "side": 256, "out": 224,
         "patch": 16, "ratio": 0.75, "bf16": False, "files": "plain"},
    ]


def _log_int(rng, lo, hi):
    return int(round(lo * (hi / lo) ** rng.random()))


def draw(rng):
    op = rng.choice(["step", "step", "step", "embed", "augment", "jpeg"])
    if op == "embed":
        patch = rng.choice([8, 12, 14, 16, 20])
        L = rng.randint(4, 16) ** 2
        return {"op": op, "B": _log_int(rng, 16, 2048), "K": max(1, int(L * rng.choice([0.15, 0.25, 0.5]))),
                "L": L, "D": 3 * patch * patch, "E": rng.choice([192, 384, 768, 1000, 1024]),
                "f32_out": rng.random() < 0.3}
    if op == "augment":
        return {"op": op, "B": _log_int(rng, 16, 2048), "side": rng.choice([256, 256, 500]),
                "stage": rng.randint(1, 3), "plus": rng.random() < 0.5,
                "patch": rng.choice([16, 16, 32]), "bf16": rng.random() < 0.5}
    patch = rng.choice([16, 16, 14, 12, 20, 32] + ([15] if op == "step" else []))
    out = patch * rng.randint((96 + patch - 1) // patch, min(16, 224 // patch))
    case = {"op": op, "B": _log_int(rng, 16, 3072), "side": 256, "out": out, "patch": patch,
            "ratio": rng.choice([0.5, 0.66, 0.75, 0.75, 0.8, 0.85]), "bf16": rng.random() < 0.5}
    if op == "jpeg":
        case["files"] = rng.choice(["rows", "plain", "indexed"])
        case["B"] = _log_int(rng, 16, 1024)
        if rng.random() < 0.3:
            case["side"], case["B"] = 500, _log_int(rng, 16, 256)
        return case
    case["side"] = rng.choice([128, 256, 256, 500])
    case["loss"] = rng.choice(["stored", "images", "none"] if patch % 2 == 0 else ["stored", "none"])
    if case["side"] == 500:
        case["B"] = min(case["B"], 1024)
    return case


# ---- inputs ------------------------------------------------------------------------------------
def _images(side, B, seed):
    """Decoded images in device memory: the shapes and the values of synth.make_images (iid bytes,
    or per channel a linear gradient and +-20 levels of noise), drawn on the device."""
    kind = KINDS[side]
    heights, widths = synth.image_shapes(kind, B, seed)
    sizes = heights.astype(np.int64) * widths
    offsets = np.zeros(B, np.int64)
    offsets[1:] = np.cumsum(3 * sizes)[:-1]
    gen = torch.Generator("cuda").manual_seed(seed)
    dev = dict(device="cuda", generator=gen)
    images = torch.empty(int(3 * sizes.sum()), dtype=torch.uint8, device="cuda")
    h = torch.from_numpy(heights).cuda()
    w = torch.from_numpy(widths).cuda()
    if kind == "uniform":
        images.random_(0, 256, generator=gen)
    else:
        base = torch.rand((B, 3), **dev) * 175 + 40
        gx = torch.rand((B, 3), **dev) * 200 - 100
        gy = torch.rand((B, 3), **dev) * 200 - 100
        for lo in range(0, B, 256):
            hi = min(B, lo + 256)
            n = torch.from_numpy(sizes[lo:hi]).cuda()
            total = int(sizes[lo:hi].sum())
            which = torch.repeat_interleave(torch.arange(lo, hi, device="cuda"), n,
                                            output_size=total)
            start = torch.cumsum(n, 0) - n
            pos = torch.arange(total, device="cuda") - start[which - lo]
            y = pos // w[which]
            x = pos - y * w[which]
            fx = (x.float() / (w[which] - 1).float() - 0.5)[:, None]
            fy = (y.float() / (h[which] - 1).float() - 0.5)[:, None]
            v = base[which] + gx[which] * fx + gy[which] * fy
            v += torch.randint(-20, 21, (total, 3), **dev)
            first = int(offsets[lo])
            images[first:first + 3 * total] = v.round_().clamp_(0, 255).to(torch.uint8).view(-1)
    return images, torch.from_numpy(offsets).cuda(), h, w


def _files(side, B, seed, restart_rows):
    """JPEG files (quality 90, 4:2:0) in device memory.  Encoding is host work, so a large batch
    holds 1024 different images, each of them several times (each time cropped differently)."""
    distinct, piece = min(B, 1024), 16
    jobs = [(min(piece, distinct - i), (seed * 1009 + i) % (1 << 31))
            for i in range(0, distinct, piece)]
    with ThreadPoolExecutor(16) as pool:
        parts = list(pool.map(lambda j: synth.make_jpegs(KINDS[side], j[0], seed=j[1],
                                                         restart_rows=restart_rows), jobs))
    files = [d[o:o + n] for d, offs, lens in parts for o, n in zip(offs, lens)]
    files = [files[b % distinct] for b in range(B)]
    sizes = np.array([f.size for f in files], np.int32)
    offsets = np.zeros(B, np.int64)
    offsets[1:] = np.cumsum(sizes.astype(np.int64))[:-1]
    return (torch.from_numpy(np.concatenate(files)).cuda(), torch.from_numpy(offsets).cuda(),
            torch.from_numpy(sizes).cuda())


def _sizes(case):
    """Training resolution, patches, values per patch, visible patches."""
    out = mae.mae_finetune_stage(mae.MAE_FINETUNE_SCHEME_1, case["stage"])[0] \
        if case["op"] == "augment" else case["out"]
    L = (out // case["patch"]) ** 2
    K = L if case["op"] == "augment" else mae.mae_num_keep(L, case["ratio"])
    return out, L, 3 * case["patch"] ** 2, K


def _prep_desc(case, state):
    return mae.make_prep_desc(*state["source"], **state["options"])


def prepare(case, seed):
    gen = torch.Generator("cuda").manual_seed(seed + 1)
    dev = dict(device="cuda", generator=gen)
    B = case["B"]
    if case["op"] == "embed":
        K, L, D, E = case["K"], case["L"], case["D"], case["E"]
        return {
            "case": case,
            # image-normalised pixel values, the ViT initialisation's weights, sine-cosine positions
            "visible": (torch.rand((B, K, D), **dev) * 4.9 - 2.2).to(torch.bfloat16),
            "ids": torch.randint(0, L, (B, K), dtype=torch.int32, **dev),
            "weight": (0.02 * torch.randn((E, D), **dev)).to(torch.bfloat16),
            "bias": 0.02 * torch.randn(E, **dev),
            "pos": torch.rand((L, E), **dev) * 2 - 1,
            "tokens": torch.empty((B, K, E), device="cuda",
                                  dtype=torch.float32 if case["f32_out"] else torch.bfloat16),
        }
    out, L, D, K = _sizes(case)
    options = dict(out_size=out, patch=case["patch"], num_keep=K, seed=seed, batch_index=1,
                   out_dtype=mae.MAE_BF16 if case["bf16"] else mae.MAE_F32,
                   max_image_side=case["side"])
    state = {"case": case, "options": options}
    if case["op"] == "jpeg":
        files, offsets, lens = _files(case["side"], B, seed, 1 if case["files"] == "rows" else 0)
        state["source"] = (files, offsets, None, None)
        options["file_sizes"] = lens
        if case["files"] == "indexed":  # once per dataset: kept with the files
            desc = _prep_desc(case, state)
            index = torch.empty(mae.mae_jpeg_index_bytes(desc), dtype=torch.uint8, device="cuda")
            space = torch.empty(mae.mae_prep_workspace_bytes(desc), dtype=torch.uint8,
                                device="cuda")
            mae.mae_jpeg_index(desc, index, space)
            options["row_index"] = index
    else:
        state["source"] = _images(case["side"], B, seed)
    if case["op"] == "augment":
        _, lo, hi, _ = mae.mae_finetune_stage(mae.MAE_FINETUNE_SCHEME_1, case["stage"])
        options["scale"] = (lo, hi)
        options["aug_mode"] = mae.MAE_AUG_THREE_PLUS if case["plus"] else mae.MAE_AUG_THREE
    desc = _prep_desc(case, state)
    want_target = case["op"] == "jpeg" or case.get("loss", "") in ("stored", "none")
    state["buf"] = mae.alloc_prep_buffers(desc, want_target=want_target)
    if case.get("loss", "none") != "none":
        pred = torch.randn((B, L, D), **dev)
        state["pred"] = pred.to(torch.bfloat16) if case["bf16"] else pred
        state["loss"] = torch.empty(1, device="cuda")
        state["grad"] = torch.empty_like(state["pred"])
        ldesc = _loss_desc(case, state, L, K)
        need = mae.mae_loss_workspace_bytes(ldesc) if case["loss"] == "stored" else \
            mae.mae_loss_from_images_workspace_bytes(desc, ldesc)
        state["space"] = torch.empty(need, dtype=torch.uint8, device="cuda")
    return state


def _loss_desc(case, state, L, K):
    return mae.make_loss_desc(state["pred"], state["buf"].target, state["buf"].mask,
                              num_masked=case["B"] * (L - K))


# ---- one pass ----------------------------------------------------------------------------------
def run(state):
    case = state["case"]
    if case["op"] == "embed":
        desc = mae.make_embed_desc(state["visible"], state["ids"], state["weight"], state["bias"],
                                   state["pos"],
                                   out_dtype=mae.MAE_F32 if case["f32_out"] else mae.MAE_BF16)
        mae.mae_patch_embed(desc, state["tokens"])
        return state["tokens"]
    desc = _prep_desc(case, state)
    buf = state["buf"]
    mae.mae_prep_batch(desc, buf.visible, buf.mask, buf.ids_restore, buf.ids_keep, buf.target,
                       buf.crop, buf.workspace)
    outputs = {"visible": buf.visible, "mask": buf.mask, "ids_restore": buf.ids_restore,
               "ids_keep": buf.ids_keep, "crop": buf.crop}
    if buf.target is not None:
        outputs["target"] = buf.target
    if case.get("loss", "none") != "none":
        options = state["options"]
        L = (options["out_size"] // options["patch"]) ** 2
        ldesc = _loss_desc(case, state, L, options["num_keep"])
        if case["loss"] == "stored":
            mae.mae_normpix_loss(ldesc, state["loss"], state["grad"], state["space"])
        else:
            mae.mae_normpix_loss_from_images(desc, buf.workspace, ldesc, state["loss"],
                                             state["grad"], state["space"])
        outputs["loss"], outputs["grad"] = state["loss"], state["grad"]
    return outputs


# ---- what a pass cannot do without -------------------------------------------------------------
def work(case):
    B = case["B"]
    if case["op"] == "embed":
        M, D, E, L = B * case["K"], case["D"], case["E"], case["L"]
        out = 4 if case["f32_out"] else 2
        return {"bytes": M * (2 * D + 4 + out * E) + 2 * E * D + 4 * E * (L + 1),
                "flops": 2 * M * D * E}
    out, L, D, K = _sizes(case)
    pixels = MEAN_PIXELS[case["side"]]
    tokens = 2 if case["bf16"] else 4
    if case["op"] == "jpeg":
        source = 0.4 * pixels  # 3.1 bits a pixel, the whole file
    else:
        source = 3 * 0.51 * pixels  # the crop: 51 % of the image on average
    per_image = source + K * D * tokens + L * (1 + 4) + 4 * K + 24
    stored = case["op"] == "jpeg" or case.get("loss", "") in ("stored", "none")
    flops = 12 * (L if stored else K) * D
    if stored:
        per_image += 4 * L * D
    if case.get("loss", "none") != "none":
        # predictions of the masked patches, the whole gradient, the mask, and the masked patches'
        # pixels from wherever they are kept
        per_image += (L - K) * D * tokens + L * D * tokens + L
        per_image += (L - K) * D * 4 if case["loss"] == "stored" else source
        flops += 10 * (L - K) * D
    return {"bytes": int(B * per_image), "flops": int(B * flops)}


def tolerance(case):
    # Whole numbers (crop boxes, masks, orders) are exact in every case.
    if case["op"] == "embed" and case["f32_out"]:
        return {"rel": 4e-6, "max": 4e-5}  # 32-bit sums of up to 1200 exact products
    if case["op"] == "embed" or case["bf16"]:
        # bf16 results are 1.7e-3 off a 64-bit evaluation; of two correct ones few values differ,
        # those on a rounding boundary, which go to either neighbour (one part in 128 at most)
        return {"rel": 1e-3, "max": 1.6e-2}
    # 32-bit interpolation, statistics and sums: 1.0e-7 .. 1.9e-7 off a 64-bit evaluation of the
    # same inputs, single values up to 1.6e-6
    return {"rel": 8e-7, "max": 8e-6}
