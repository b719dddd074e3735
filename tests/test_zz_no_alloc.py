"""qrm_detect_static (the entry point that allocates nothing) against qrm_detect, through the C ABI."""
import numpy as np
import pytest
import torch

import oracle
import synth
from gpu_util import dev, empty, check_logits

pytestmark = pytest.mark.gpu


def outputs(cfg, N):
    return (empty((N, cfg.n_bits), torch.float32), empty((N, cfg.n_bits), torch.uint8), empty((N, cfg.k), torch.uint8),
            empty((N, cfg.n), torch.uint8), empty((N,), torch.int8))


def test_detect_static_equals_detect_on_two_calls_in_a_row():
    """Two calls in a row on the shared static workspace, the second with a smaller input (fewer images, and then a
    smaller tile shape): same bytes out as qrm_detect with the same micro-batch; the first call also against the
    oracle.  Sizes beyond the array are refused."""
    import paper_2509_02447_amd as q
    cfg = synth.CONFIGS["C2"]
    wts = synth.config_weights(cfg)
    ctx = q.Context(weights=wts, rs=dict(m=cfg.m, prim_poly=cfg.prim_poly, n=cfg.n, k=cfg.k, fcr=cfg.fcr))
    ref_ctx = q.Context(weights=wts, rs=dict(m=cfg.m, prim_poly=cfg.prim_poly, n=cfg.n, k=cfg.k, fcr=cfg.fcr))
    for call, (N, start) in enumerate(((150, 0), (37, 400))):     # 150 images = three micro-batches of the array's 56
        imgs = synth.images(cfg, start, N)
        imgs[1::7] = synth.field_images(cfg, start, len(imgs[1::7]))
        off = synth.offsets(cfg, start, N)
        d_img, d_off = dev(imgs), dev(off)
        a, b = outputs(cfg, N), outputs(cfg, N)
        ctx.qrm_detect_static(d_img, N, cfg.H, cfg.W, d_off, cfg.tile, *a)
        ref_ctx.qrm_detect(d_img, N, cfg.H, cfg.W, d_off, cfg.tile, *b)
        torch.cuda.synchronize()
        names = ("logits", "bits", "msg", "codeword", "nerr")
        for name, x, y in zip(names, a, b):
            assert np.array_equal(x.cpu().numpy(), y.cpu().numpy()), (call, name)
        if call == 0:
            sample = [0, 1, 8, 55, 56, 57, 111, 112, 149]
            flat = np.array([i % 7 == 1 and bool(synth.field_is_flat(cfg, start, N)[i // 7]) for i in sample])
            ref = oracle.detect(wts, imgs[sample], off[sample], cfg.tile, cfg.m, cfg.prim_poly, cfg.n, cfg.k, cfg.fcr)
            check_logits(a[0].cpu().numpy()[sample], ref["logits"], a[1].cpu().numpy()[sample], what="qrm_detect_static", flat=flat)
            syms = oracle.bits_to_symbols(a[1].cpu().numpy(), cfg.m)
            om, oc, oe = oracle.rs_decode(syms, cfg.m, cfg.prim_poly, cfg.n, cfg.k, cfg.fcr)
            assert np.array_equal(a[2].cpu().numpy(), om) and np.array_equal(a[3].cpu().numpy(), oc)
            assert np.array_equal(a[4].cpu().numpy(), oe)
    # a third call with a smaller tile (other layout of the same array), optional outputs left out
    N, tile = 9, 32
    imgs, off = synth.images(cfg, 900, N), synth.offsets(cfg, 900, N) // 2
    d_img, d_off = dev(imgs), dev(off)
    m1, e1, m2, e2 = empty((N, cfg.k), torch.uint8), empty((N,), torch.int8), empty((N, cfg.k), torch.uint8), empty((N,), torch.int8)
    ctx.qrm_detect_static(d_img, N, cfg.H, cfg.W, d_off, tile, None, None, m1, None, e1)
    ref_ctx.qrm_detect(d_img, N, cfg.H, cfg.W, d_off, tile, None, None, m2, None, e2)
    torch.cuda.synchronize()
    assert np.array_equal(m1.cpu().numpy(), m2.cpu().numpy()) and np.array_equal(e1.cpu().numpy(), e2.cpu().numpy())
    # beyond the array: one 640 x 640 tile needs 2 x 50 MiB of activations
    big = empty((1, 3, 640, 640), torch.uint8)
    with pytest.raises(q.QrmError) as e:
        ctx.qrm_detect_static(big, 1, 640, 640, None, 640, None, None, m1, None, e1)
    assert e.value.status == q.QRM_E_UNSUPPORTED and "static workspace" in e.value.message
    ctx.qrm_detect_static(d_img, 0, cfg.H, cfg.W, d_off, tile, None, None, m1, None, e1)      # N == 0: no-op
    ctx.close()
    ref_ctx.close()


@pytest.mark.parametrize("tile,n_blocks", [(305, 8), (308, 3), (502, 2)])
def test_detect_static_takes_tiles_up_to_the_size_of_its_array(tile, n_blocks):
    """Tiles of 64 channels, the last of them the largest whose activations fit the array one image at a time; same bytes
    as qrm_detect with the same micro-batch."""
    import paper_2509_02447_amd as q
    cfg = synth.CONFIGS["C2"]
    wts = synth.extractor_weights(3, n_blocks, 64, cfg.n_bits, seed_index=tile)
    rs = dict(m=cfg.m, prim_poly=cfg.prim_poly, n=cfg.n, k=cfg.k, fcr=cfg.fcr)
    ctx, ref_ctx = q.Context(weights=wts, rs=rs), q.Context(weights=wts, rs=rs)
    N = 2 if tile < 400 else 1
    d_img = dev(np.random.default_rng(tile).integers(0, 256, size=(N, 3, tile, tile), dtype=np.uint8))
    a, b = outputs(cfg, N), outputs(cfg, N)
    ctx.qrm_detect_static(d_img, N, tile, tile, None, tile, *a)
    ref_ctx.qrm_detect(d_img, N, tile, tile, None, tile, *b)
    torch.cuda.synchronize()
    for name, x, y in zip(("logits", "bits", "msg", "codeword", "nerr"), a, b):
        assert np.array_equal(x.cpu().numpy(), y.cpu().numpy()), name
    ctx.close()
    ref_ctx.close()
