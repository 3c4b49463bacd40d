"""End-to-end parity of the HIP recovery path (through the C ABI) against the
FP64 oracle, plus the serving semantics of the paper's receiver: clean frames
become references, recovered frames never do, the same references serve later
targets through the temporal-distance embedding (Sec. 3.4.1)."""
import numpy as np
import pytest

import oracle
import synth
from tests.gpu_util import check_received_and_codes, compare, push_refs, recover

pytestmark = pytest.mark.gpu

FP32, BF16 = 0, 1
SMALL = dict(enc_depth=2, dec_depth=1)


def _rec(blobs, prec, **kw):
    from paper_2604_27441_amd import Recoverer
    kw.setdefault("max_batch_tokens", 8192)
    return Recoverer(blobs[0], blobs[1], precision=prec, **kw)


@pytest.fixture(scope="module")
def c1():
    req = synth.make_batch("c1")[0]
    blobs = synth.make_weights(0)
    ref = oracle.recover(req, blobs)
    return req, blobs, ref


@pytest.fixture(scope="module")
def c1_bf16_budget(c1):
    """Error of the BF16-rounding oracle against the exact one: the budget the
    BF16 kernels are held to (twice its MSE, four times its max error)."""
    req, blobs, ref = c1
    emu = oracle.recover(req, blobs, rnd=oracle.Rounding(oracle.bf16_round))
    gpu_like = {"rgb_f": emu["rgb"][1], "depth_f": emu["depth"][1]}
    return compare(req, gpu_like, ref)


def test_c1_fp32_parity(c1):
    req, blobs, ref = c1
    with _rec(blobs, FP32) as rec:
        push_refs(rec, 0, req)
        out = recover(rec, [(0, req)])[0]
    assert out["completion"].status == 0
    check_received_and_codes(req, out)
    e = compare(req, out, ref)
    print("c1 fp32", e)
    assert e["rgb_psnr"] >= 80.0, e
    assert e["depth_maxabs"] <= 0.5, e


def test_c1_bf16_parity(c1, c1_bf16_budget):
    req, blobs, ref = c1
    with _rec(blobs, BF16) as rec:
        push_refs(rec, 0, req)
        out = recover(rec, [(0, req)])[0]
    check_received_and_codes(req, out)
    e = compare(req, out, ref)
    b = c1_bf16_budget
    print("c1 bf16", e, "budget", b)
    assert e["rgb_psnr"] >= 45.0, e
    assert e["rgb_psnr"] >= b["rgb_psnr"] - 3.02, (e, b)          # MSE <= 2x the rounding oracle's
    assert e["depth_rms_lost"] <= np.sqrt(2.0) * b["depth_rms_lost"], (e, b)
    assert e["depth_maxabs"] <= 4.0 * b["depth_maxabs"], (e, b)


def _small(prec, req, k=5, T=2, n_ref=None, blobs=None, **kw):
    blobs = blobs or synth.make_weights(3, tubelet=T, perturb_seed=4, **SMALL)
    refs = {}
    ref = None
    with _rec(blobs, prec, k=k, tubelet=T, **SMALL, **kw) as rec:
        push_refs(rec, 0, req, n_ref=n_ref)
        out = recover(rec, [(0, req)])[0]
    r2 = dict(req)
    if n_ref is not None:
        for key in ("rgb_refs", "depth_refs", "ref_idx"):
            r2[key] = req[key][len(req["ref_idx"]) - n_ref:]
    ref = oracle.recover(r2, blobs, k=k, tubelet=T, **SMALL)
    return out, ref


@pytest.mark.parametrize("H,W", [(16, 16), (40, 56), (20, 36), (192, 256), (100, 30)])
def test_ragged_sizes_fp32(H, W):
    req = synth.make_request(31, 32, H, W, loss=("stripes", 0.5))
    out, ref = _small(FP32, req)
    check_received_and_codes(req, out)
    e = compare(req, out, ref)
    assert e["rgb_maxabs"] <= 1e-4 and e["depth_maxabs"] <= 0.5, e


@pytest.mark.parametrize("k,T,n_ref", [(5, 2, 2), (4, 2, None), (5, 3, None), (3, 1, None), (7, 2, 5), (7, 3, None),
                                       (6, 3, 4), (1, 2, None), (1, 1, None), (2, 3, None)])
def test_history_and_tubelet_variants(k, T, n_ref):
    req = synth.make_request(41, 42, 48, 64, k=k, loss=("stripes", 0.5))
    out, ref = _small(FP32, req, k=k, T=T, n_ref=n_ref)
    e = compare(req, out, ref)
    assert e["rgb_maxabs"] <= 1e-4 and e["depth_maxabs"] <= 0.5, e


def test_raw_prediction_without_composite():
    req = synth.make_request(51, 52, 48, 64, loss=("stripes", 0.5))
    out, ref = _small(FP32, req, composite=0)
    assert np.abs(out["rgb_f"] - np.clip(ref["rgb"][0], 0, 1)).max() <= 1e-4
    assert np.abs(out["depth_f"] - np.clip(4000 * ref["depth"][0][..., 0], 0, 65535)).max() <= 0.5


def test_batch_invariance_and_host_pointers():
    """A request gives the same bytes alone and inside a mixed batch of other
    streams and resolutions, and through host or device pointers."""
    blobs = synth.make_weights(3, perturb_seed=4, **SMALL)
    reqs = [synth.make_request(61 + i, 62 + i, H, W, loss=("stripes", 0.4))
            for i, (H, W) in enumerate([(48, 64), (40, 56), (96, 128), (20, 36)])]
    for prec in (FP32, BF16):
        with _rec(blobs, prec, **SMALL) as rec:
            for s, r in enumerate(reqs):
                push_refs(rec, s, r)
            mixed = recover(rec, list(enumerate(reqs)))
            alone = [recover(rec, [(s, r)])[0] for s, r in enumerate(reqs)]
            host = recover(rec, [(2, reqs[2])], device_ptrs=False)[0]
        for a, b in zip(mixed, alone):
            for key in ("rgb", "depth", "rgb_f", "depth_f"):
                assert np.array_equal(a[key], b[key]), key
        for key in ("rgb", "depth", "rgb_f", "depth_f"):
            assert np.array_equal(host[key], alone[2][key]), key


@pytest.mark.parametrize("prec,n", [(BF16, 5), (BF16, 20), (2, 5), (2, 20), (FP32, 2), (FP32, 4), (FP32, 8)])
def test_batches_that_take_other_tile_forms(prec, n):
    """A 256 x 192 request (576 tokens) alone and beside n - 1 others, whose
    rows together take other tile forms of the products, the Q / K / V split
    and transposed V with them: BF16 64 x 64 alone, 128 x 128 at 5 and 256 x 64
    (decoder) at 20, FP8 64 x 64, 128 x 64 and 128 x 128.  Those give the same
    bits.  The FP32 forms sum K in four groups, two or one, by the rows of the
    whole batch, so a request's FP32 result depends on its batch, by rounding
    alone: no further apart than twice what either may be from the oracle."""
    import torch
    from tests.gpu_util import dev
    blobs = synth.make_weights(3, perturb_seed=4, enc_depth=1, dec_depth=1)
    req = synth.make_request(121, 122, 192, 256, loss=("stripes", 0.4))
    other = synth.make_request(123, 124, 192, 256, loss=("stripes", 0.4))
    cap = 20 * 576
    big = synth.make_request(125, 126, 768, 1280, loss=("stripes", 0.4))   # 11520 tokens, a whole batch

    def buffers(r):
        h, w = r["height"], r["width"]
        return ([dev(r["rgb"]), dev(r["mask_rgb"]), dev(r["depth"]), dev(r["mask_depth"])],
                dict(rgb=torch.zeros((h, w, 3), dtype=torch.uint8, device="cuda"),
                     depth=torch.zeros((h, w), dtype=torch.int16, device="cuda"),
                     rgb_f=torch.zeros((h, w, 3), device="cuda"), depth_f=torch.zeros((h, w), device="cuda")))

    with _rec(blobs, prec, enc_depth=1, dec_depth=1, max_batch=24, max_batch_tokens=cap) as rec:
        if prec == 2:
            push_refs(rec, 30, req)
            rec.calibrate(1)
            recover(rec, [(30, req)])
            rec.calibrate(0)
        push_refs(rec, 40, big)
        # the small requests queue behind whole batches and then go together
        items = [(40, big)] * 8 + [(s, other if s else req) for s in range(n)]
        for s in range(n):
            push_refs(rec, s, other if s else req)
        bufs = [buffers(r) for _, r in items]
        torch.cuda.synchronize()
        batches = rec.stats()["batches"]
        tickets = [rec.submit(s, int(r["t_target"]), r["width"], r["height"], rgb=i[0], mask_rgb=i[1], depth=i[2],
                              mask_depth=i[3], rgb_out=o["rgb"], depth_out=o["depth"], rgb_out_f32=o["rgb_f"],
                              depth_out_f32=o["depth_f"], device_ptrs=True) for (s, r), (i, o) in zip(items, bufs)]
        assert all(c.status == 0 for c in rec.wait(tickets).values())
        assert rec.stats()["batches"] == batches + 9
        mixed = {k: v.cpu().numpy() for k, v in bufs[8][1].items()}
        mixed["depth"] = mixed["depth"].view(np.uint16)
        alone = recover(rec, [(0, req)])[0]
    if prec != FP32:
        for key in ("rgb", "depth", "rgb_f", "depth_f"):
            assert np.array_equal(mixed[key], alone[key]), key
    else:
        assert np.abs(mixed["rgb_f"] - alone["rgb_f"]).max() <= 2e-4
        assert np.abs(mixed["depth_f"] - alone["depth_f"]).max() <= 1.0


def test_references_reused_across_later_targets():
    """Two corrupted frames in a row use the same clean references; the second
    one sees a larger temporal distance (no recovered frame enters the ring)."""
    blobs = synth.make_weights(3, perturb_seed=4, **SMALL)
    req = synth.make_request(71, 72, 48, 64, loss=("stripes", 0.5))
    later = dict(req)
    later["t_target"] = req["t_target"] + 2
    with _rec(blobs, FP32, **SMALL) as rec:
        push_refs(rec, 0, req)
        a = recover(rec, [(0, req)])[0]
        b = recover(rec, [(0, later)])[0]
    ra = oracle.recover(req, blobs, **SMALL)
    rb = oracle.recover(later, blobs, **SMALL)
    assert compare(req, a, ra)["rgb_maxabs"] <= 1e-4
    assert compare(later, b, rb)["rgb_maxabs"] <= 1e-4


def test_clean_frame_copy_and_resolution_change():
    blobs = synth.make_weights(3, **SMALL)
    req = synth.make_request(81, 82, 32, 48, loss=("stripes", 0.5))
    with _rec(blobs, BF16, **SMALL) as rec:
        # a clean frame comes back unchanged
        clean = dict(req)
        clean["mask_rgb"] = np.zeros_like(req["mask_rgb"])
        clean["mask_depth"] = np.zeros_like(req["mask_depth"])
        push_refs(rec, 5, req)
        out = recover(rec, [(5, clean)])[0]
        assert np.array_equal(out["rgb"], req["rgb"]) and np.array_equal(out["depth"], req["depth"])
        # a resolution change starts a new reference set: one clean frame at
        # the new size serves (repeated as the oldest, k - 1 times)
        other = synth.make_request(83, 84, 48, 64, loss=("stripes", 0.5))
        push_refs(rec, 5, other, n_ref=1)
        out = recover(rec, [(5, other)])[0]
        assert out["completion"].status == 0
    r1 = dict(other)
    for key in ("rgb_refs", "depth_refs", "ref_idx"):
        r1[key] = other[key][-1:]
    ref = oracle.recover(r1, blobs, **SMALL)
    e = compare(other, out, ref)
    assert e["rgb_psnr"] >= 40, e


@pytest.mark.parametrize("loss", [0.10, 0.30, 0.50])
def test_c2_640x480_fp32_parity(loss):
    """640x480, one pair, Gilbert-Elliott slice loss at mean 10/30/50 %, full
    12 + 4 block model, FP32 form against the FP64 oracle."""
    req = synth.make_request(1002, 2002, 480, 640, loss=("ge", loss))
    blobs = synth.make_weights(0)
    with _rec(blobs, FP32) as rec:
        push_refs(rec, 0, req)
        out = recover(rec, [(0, req)])[0]
    ref = oracle.recover(req, blobs)
    check_received_and_codes(req, out)
    e = compare(req, out, ref)
    print(f"c2 fp32 L={loss}", e)
    assert e["rgb_psnr"] >= 80.0, e
    assert e["depth_maxabs"] <= 0.5, e


def test_graph_replays_match_eager():
    """Graph-captured launches (one graph per capacity bucket) reproduce the
    eager launches bit for bit on every replay, with eager work between."""
    blobs = synth.make_weights(3, perturb_seed=4, **SMALL)
    reqs = [synth.make_request(91 + i, 92 + i, H, W, loss=("stripes", 0.4))
            for i, (H, W) in enumerate([(48, 64), (40, 56), (96, 128), (20, 36)])]
    rounds = [[0, 1, 2, 3], [2], [1, 3], [0, 1, 2, 3], [3], [0, 2]]
    with _rec(blobs, BF16, **SMALL) as rec:
        for s, r in enumerate(reqs):
            push_refs(rec, s, r)
        eager = {s: recover(rec, [(s, reqs[s])])[0] for s in range(4)}
    with _rec(blobs, BF16, graphs=True, **SMALL) as rec:
        for s, r in enumerate(reqs):
            push_refs(rec, s, r)
        for rnd in rounds:
            outs = recover(rec, [(s, reqs[s]) for s in rnd])
            for s, o in zip(rnd, outs):
                for key in ("rgb", "depth", "rgb_f", "depth_f"):
                    assert np.array_equal(o[key], eager[s][key]), (rnd, s, key)
            # eager device work and a synchronisation between replays
            import torch
            torch.ones(1 << 20, device="cuda").sum().item()


def test_fp8_graph_replays_match_eager():
    """The FP8 form (E4M3 block products and attention with calibrated scales)
    captured in graphs reproduces its eager launches bit for bit, both
    contexts calibrated on the same frames."""
    FP8 = 2
    blobs = synth.make_weights(3, perturb_seed=4, **SMALL)
    reqs = [synth.make_request(191 + i, 192 + i, H, W, loss=("stripes", 0.4))
            for i, (H, W) in enumerate([(48, 64), (40, 56), (96, 128)])]
    calib = [synth.make_request(10000 + i, 10100 + i, 48, 64, loss=("ge", 0.3)) for i in range(3)]
    rounds = [[0, 1, 2], [2], [0, 1], [1, 2]]

    def ctx(**kw):
        rec = _rec(blobs, FP8, **SMALL, **kw)
        for s, r in enumerate(reqs):
            push_refs(rec, s, r)
        for s, r in enumerate(calib):
            push_refs(rec, 10 + s, r)
        rec.calibrate(1)
        recover(rec, [(10 + s, r) for s, r in enumerate(calib)])
        rec.calibrate(0)
        return rec

    rec = ctx()
    try:
        eager = {s: recover(rec, [(s, reqs[s])])[0] for s in range(len(reqs))}
    finally:
        rec.close()
    rec = ctx(graphs=True)
    try:
        for rnd in rounds:
            outs = recover(rec, [(s, reqs[s]) for s in rnd])
            for s, o in zip(rnd, outs):
                assert o["completion"].status == 0
                for key in ("rgb", "depth", "rgb_f", "depth_f"):
                    assert np.array_equal(o[key], eager[s][key]), (rnd, s, key)
            import torch
            torch.ones(1 << 20, device="cuda").sum().item()
    finally:
        rec.close()


def test_many_batches_in_flight():
    """Requests submitted back to back (several batches queued and in flight
    on the GPU) give the same bytes as each request run alone."""
    import torch
    from paper_2604_27441_amd import Recoverer
    blobs = synth.make_weights(3, perturb_seed=4, **SMALL)
    reqs = [synth.make_request(101 + i, 102 + i, 48, 64, loss=("stripes", 0.5)) for i in range(4)]
    with _rec(blobs, BF16, graphs=True, max_batch=2, **SMALL) as rec:
        for s, r in enumerate(reqs):
            push_refs(rec, s, r)
        alone = {s: recover(rec, [(s, reqs[s])])[0] for s in range(4)}
        outs, tickets = [], []
        for rep in range(3):
            for s, r in enumerate(reqs):
                o = torch.zeros((48, 64, 3), dtype=torch.uint8, device="cuda")
                od = torch.zeros((48, 64), dtype=torch.int16, device="cuda")
                t = rec.submit(s, int(r["t_target"]), 64, 48, rgb=torch.from_numpy(r["rgb"]).cuda(),
                               mask_rgb=torch.from_numpy(r["mask_rgb"]).cuda(),
                               depth=torch.from_numpy(r["depth"]).cuda(),
                               mask_depth=torch.from_numpy(r["mask_depth"]).cuda(),
                               rgb_out=o, depth_out=od, device_ptrs=True)
                outs.append((s, o, od))
                tickets.append(t)
        got = rec.wait(tickets)
        assert all(c.status == 0 for c in got.values())
        for s, o, od in outs:
            assert np.array_equal(o.cpu().numpy(), alone[s]["rgb"])
            assert np.array_equal(od.cpu().numpy().view(np.uint16), alone[s]["depth"])


def test_fp8_form_against_rounding_oracle():
    """FP8 form: after a calibration pass over seeded frames (run by the
    library and, independently, by the oracle on the same frames), the GPU's
    error against FP64 stays within the FP8-rounding oracle's error budget
    (twice its MSE, four times its max error); received pixels stay exact."""
    FP8 = 2
    blobs = synth.make_weights(3, perturb_seed=4, **SMALL)
    target = synth.make_request(111, 112, 96, 128, loss=("stripes", 0.5))
    calib = [synth.make_request(10000 + i, 10100 + i, 96, 128, loss=("ge", 0.3)) for i in range(4)]
    scales = {}
    for mod in ("rgb", "depth"):
        rec = oracle.AbsMaxRecorder()
        for r in calib:
            oracle.recover(r, blobs, rnd=rec, modalities=(mod,), **SMALL)
        scales[mod] = rec.scales()
    exact = oracle.recover(target, blobs, **SMALL)
    emu = {}
    for mod in ("rgb", "depth"):
        emu.update(oracle.recover(target, blobs, rnd=oracle.FP8Rounding(scales[mod]), modalities=(mod,), **SMALL))
    with _rec(blobs, FP8, **SMALL) as rec:
        for s, r in enumerate(calib):
            push_refs(rec, s, r)
        push_refs(rec, 9, target)
        before = recover(rec, [(9, target)])[0]          # uncalibrated: computes as BF16
        rec.calibrate(1)
        recover(rec, list(enumerate(calib)))
        rec.calibrate(0)
        out = recover(rec, [(9, target)])[0]
    check_received_and_codes(target, out)
    assert not np.array_equal(out["rgb_f"], before["rgb_f"])
    e = compare(target, out, exact)
    b = compare(target, {"rgb_f": emu["rgb"][1], "depth_f": emu["depth"][1]}, exact)
    print("fp8", e, "budget", b)
    assert e["rgb_psnr"] >= b["rgb_psnr"] - 3.02, (e, b)
    assert e["depth_rms_lost"] <= np.sqrt(2.0) * b["depth_rms_lost"], (e, b)
    assert e["depth_maxabs"] <= 4.0 * b["depth_maxabs"], (e, b)


@pytest.mark.parametrize("prec", [FP32, BF16])
def test_mask_without_lost_pixels_returns_the_input(prec):
    """A frame that goes through recovery but lost nothing comes back as it
    arrived, byte for byte (every pixel is a received pixel)."""
    req = synth.make_request(91, 92, 40, 56, loss=("none", 0))
    assert not req["mask_rgb"].any() and not req["mask_depth"].any()
    out, _ = _small(prec, req)
    assert out["completion"].status == 0
    check_received_and_codes(req, out)
    assert np.array_equal(out["rgb"], req["rgb"]) and np.array_equal(out["depth"], req["depth"])


def test_everything_lost_fp32():
    """A frame with every slice lost: the network sees the references and an
    all-zero target, and every output pixel is the clamped prediction."""
    req = synth.make_request(93, 94, 40, 56, loss=("all", 0))
    assert req["mask_rgb"].all() and req["mask_depth"].all()
    out, ref = _small(FP32, req)
    check_received_and_codes(req, out)
    e = compare(req, out, ref)
    assert e["rgb_maxabs"] <= 1e-4 and e["depth_maxabs"] <= 0.5, e


def test_modalities_keep_separate_rings():
    """RGB lost while the depth of the same frame arrived intact: the RGB is
    recovered, the depth is copied and becomes the newest depth reference.
    The next frame's depth recovery then uses it, while the RGB references
    stay as they were (Sec. 3.4.2: separate models and losses per modality)."""
    import torch
    from tests.gpu_util import dev
    blobs = synth.make_weights(3, perturb_seed=4, **SMALL)
    H, W = 40, 56
    req = synth.make_request(95, 98, H, W, loss=("stripes", 0.5))
    nxt = synth.make_request(95, 97, H, W, t_target=req["t_target"] + 1, loss=("stripes", 0.5))
    assert req["mask_rgb"].any() and nxt["mask_depth"].any()

    def outs():
        return dict(rgb=torch.zeros((H, W, 3), dtype=torch.uint8, device="cuda"),
                    depth=torch.zeros((H, W), dtype=torch.int16, device="cuda"),
                    rgb_f=torch.zeros((H, W, 3), dtype=torch.float32, device="cuda"),
                    depth_f=torch.zeros((H, W), dtype=torch.float32, device="cuda"))

    def run(rec, r, rgb_lost):
        o = outs()
        ins = [dev(r["rgb"]), dev(r["mask_rgb"]), dev(r["depth"]), dev(r["mask_depth"])]
        t = rec.submit(0, int(r["t_target"]), W, H, rgb=ins[0], mask_rgb=ins[1] if rgb_lost else None,
                       depth=ins[2], mask_depth=None if rgb_lost else ins[3], rgb_out=o["rgb"], depth_out=o["depth"],
                       rgb_out_f32=o["rgb_f"], depth_out_f32=o["depth_f"], device_ptrs=True)
        c = rec.wait([t])[t]
        assert c.status == 0, c
        got = {k: v.cpu().numpy() for k, v in o.items()}
        got["depth"] = got["depth"].view(np.uint16)
        return got

    with _rec(blobs, FP32, **SMALL) as rec:
        push_refs(rec, 0, req)
        a = run(rec, req, rgb_lost=True)
        b = run(rec, nxt, rgb_lost=False)
    ra = oracle.recover(req, blobs, modalities=("rgb",), **SMALL)["rgb"]
    assert np.abs(a["rgb_f"] - ra[1]).max() <= 1e-4
    assert np.array_equal(a["depth"], req["depth"])                      # copied as received
    r2 = dict(nxt)
    r2["depth_refs"] = list(req["depth_refs"][1:]) + [req["depth"]]        # newest depth reference
    r2["ref_idx"] = list(req["ref_idx"][1:]) + [req["t_target"]]
    rb = oracle.recover(r2, blobs, modalities=("depth",), **SMALL)["depth"]
    assert np.abs(b["depth_f"] - rb[1]).max() <= 0.5
    assert np.array_equal(b["rgb"], nxt["rgb"])
    # the same depth with the old references differs: the ring really moved
    r_old = oracle.recover(nxt, blobs, modalities=("depth",), **SMALL)["depth"]
    lost = nxt["mask_depth"] != 0
    assert np.abs(r_old[1] - rb[1])[lost].max() > 1.0
