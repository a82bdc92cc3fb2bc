"""GPU parity: the HIP path, called through the C ABI, against the CPU oracle
on the same seeded inputs.  Bars: index sets bit-exact except counted near-ties
(relative gap < 1e-6 in the oracle's own fp32 scores); merged bf16 features
within 1e-3 + 2e-3 |o| of the oracle's unrounded value and within 0.52 bf16 ulp;
retention within 1e-5."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

from oracle import rtprune_oracle as orc  # noqa: E402
from paper_2605_00392_amd import rtprune as rt  # noqa: E402
from paper_2605_00392_amd import synth  # noqa: E402
from tests import harness as hz  # noqa: E402


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    rt.load_library()          # raises if the HIP library is missing: no fallback


def _log(rep, name):
    print(f"\n[{name}] images={rep.images} ratio_boundary={rep.ratio_boundary} "
          f"sel_near_ties={rep.selection_near_ties} pair_near_ties={rep.pairing_near_ties}/{rep.pairs_checked} "
          f"max_ratio_err={rep.max_ratio_err:.2e} max_row_rel={rep.max_merge_row_rel:.2e} "
          f"max_plan_rel={rep.max_plan_rel:.2e} max_score_abs={rep.max_score_abs:.2e}", flush=True)
    for n in rep.notes:
        print("   ", n, flush=True)


def _assert_fused_equals_staged(f, s, batch):
    np.testing.assert_array_equal(f["keep"], s["keep"])
    np.testing.assert_array_equal(f["out_offsets"], s["out_offsets"])
    np.testing.assert_array_equal(f["sel"], s["sel"])
    np.testing.assert_array_equal(f["pair"], s["pair"])
    n_out = int(s["out_offsets"][-1])
    np.testing.assert_array_equal(f["out"][:n_out], s["out"][:n_out])


# ------------------------------------------------------------- the five workloads
def test_c1_single_image_fp32():
    batch = synth.gen_batch(1)
    f = hz.run_prune(batch)
    assert f["rc"] == 0 and f["status"] == 0
    assert list(f["keep"]) == [54]
    _log(hz.compare_batch(batch, f), "c1 fused")
    s = hz.run_staged(batch)
    _log(hz.compare_batch(batch, s, staged=True), "c1 staged")
    _assert_fused_equals_staged(f, s, batch)


def test_c2_batch32_256tok_bf16():
    batch = synth.gen_batch(2)
    f = hz.run_prune(batch)
    assert f["rc"] == 0 and f["status"] == 0
    assert (f["keep"] == 216).all()
    _log(hz.compare_batch(batch, f), "c2 fused")
    s = hz.run_staged(batch)
    _log(hz.compare_batch(batch, s, staged=True), "c2 staged")
    _assert_fused_equals_staged(f, s, batch)


def test_c3_batch64_400tok_dynamic():
    batch = synth.gen_batch(3)
    f = hz.run_prune(batch)
    assert f["rc"] == 0 and f["status"] == 0
    _log(hz.compare_batch(batch, f), "c3 fused")
    s = hz.run_staged(batch)
    _log(hz.compare_batch(batch, s, staged=True), "c3 staged")
    _assert_fused_equals_staged(f, s, batch)


def test_c3_affine_normalisation_hits_the_clamp():
    # f_normalize with (lo, hi) = (0, 0.05): larger pruned sets, some images at the 0.6 clamp
    batch = synth.gen_batch(3, images=range(16))
    params = dict(batch.params, phi_lo=0.0, phi_hi=0.05)
    f = hz.run_prune(batch, params)
    assert f["rc"] == 0 and f["status"] == 0
    rep = hz.compare_batch(batch, f, params)
    _log(rep, "c3 phi_hi=0.05")
    assert (f["ratio"] == np.float32(0.6)).any() and f["ratio"].max() > 0.6


def _log_counts(rep, name):
    """The whole-batch counts the parity clause asks to be reported."""
    print(f"[{name}] WHOLE BATCH: images compared={rep.images} ratio-boundary images={rep.ratio_boundary} "
          f"selection near-ties={rep.selection_near_ties} pairing near-ties={rep.pairing_near_ties} "
          f"of {rep.pairs_checked} pairing columns", flush=True)


def test_c4_ragged_multi_tile():
    batch = synth.gen_batch_parallel(4)
    assert batch.batch == 128 and batch.max_tokens <= 1156
    f = hz.run_prune(batch)
    assert f["rc"] == 0 and f["status"] == 0
    rep = hz.compare_batch_parallel(batch, f, chunk=4)            # every image
    _log(rep, "c4 fused (all 128 images)")
    _log_counts(rep, "c4")
    assert rep.images == 128
    picks = list(range(0, 128, 6))
    sub = synth.subset(batch, picks[:6])
    s = hz.run_staged(sub)
    _log(hz.compare_batch(sub, s, staged=True), "c4 staged subset")
    # a ragged batch equals each image alone
    alone = hz.run_prune(synth.subset(batch, [picks[3]]))
    b = picks[3]
    o0, o1 = int(f["out_offsets"][b]), int(f["out_offsets"][b + 1])
    np.testing.assert_array_equal(alone["out"][: o1 - o0], f["out"][o0:o1])


def test_c5_full_batch_against_oracle():
    batch = synth.gen_batch_parallel(5)
    assert batch.batch == 1024 and batch.total_tokens == 409600
    f = hz.run_prune(batch)
    assert f["rc"] == 0 and f["status"] == 0
    g = hz.run_prune(batch)                                       # run-to-run determinism
    np.testing.assert_array_equal(f["out"], g["out"])
    np.testing.assert_array_equal(f["pair"], g["pair"])
    del g
    rep = hz.compare_batch_parallel(batch, f)                     # every image
    _log(rep, "c5 fused (all 1024 images)")
    _log_counts(rep, "c5")
    assert rep.images == 1024
    keep = f["keep"].astype(np.int64)
    assert (np.diff(f["out_offsets"].astype(np.int64)) == keep).all()
    assert (keep >= np.ceil(0.6 * 400 - 1e-3)).all() and (keep <= 400).all()


def test_c9_full_batch_against_oracle():
    """The benchmark's pages at the paper's average retention (Table 2), whole batch: 63 pruned
    tokens per page, enough pages for the matrix-core merge kernel of the middling pruned sets
    to run by default."""
    batch = synth.gen_batch_parallel(9)
    assert batch.batch == 1024 and batch.total_tokens == 409600
    f = hz.run_prune(batch)
    assert f["rc"] == 0 and f["status"] == 0
    assert (f["keep"] == 337).all()
    g = hz.run_prune(batch)
    np.testing.assert_array_equal(f["out"], g["out"])
    del g
    rep = hz.compare_batch_parallel(batch, f)                     # every image
    _log(rep, "c9 fused (all 1024 images)")
    _log_counts(rep, "c9")
    assert rep.images == 1024 and rep.pairs_checked == 1024 * 63


def test_c6_full_batch_against_oracle():
    """The 1083-token pages (Table 6: 560 kept), whole batch in the benchmark's launch
    configuration: 64 images on the 64 four-workgroup slots of the kernel that keeps their
    Sinkhorn matrices on chip, every image compared."""
    batch = synth.gen_batch_parallel(6)
    assert batch.batch == 64 and batch.max_tokens == 1083
    f = hz.run_prune(batch)
    assert f["rc"] == 0 and f["status"] == 0
    assert (f["keep"] == 560).all()
    rep = hz.compare_batch_parallel(batch, f, chunk=2)            # every image
    _log(rep, "c6 fused (all 64 images)")
    _log_counts(rep, "c6")
    assert rep.images == 64 and rep.pairs_checked == 64 * 523


# ------------------------------------------- other OCR models' token counts (Table 6)
@pytest.mark.parametrize("cfg,images,kept", [(6, 3, 560), (7, 2, 1238), (8, 1, 2783), (9, 6, 337)])
def test_large_pages(cfg, images, kept):
    batch = synth.gen_batch(cfg, images=range(images))
    f = hz.run_prune(batch)
    assert (f["keep"] == kept).all()
    rep = hz.compare_batch(batch, f, staged=False)
    _log(rep, f"c{cfg} {images} image(s)")
    s = hz.run_staged(batch)
    rows = int(s["out_offsets"][-1])
    np.testing.assert_array_equal(f["out"][:rows], s["out"][:rows])
    np.testing.assert_array_equal(f["pair"], s["pair"])
    # the staged results carry the scores and the plan: compared entry by entry
    rep2 = hz.compare_batch(batch, s, staged=True)
    _log(rep2, f"c{cfg} staged")
    assert rep2.max_score_abs <= hz.SCORE_ATOL


def _clustered(counts, d, dtype, seed, **params):
    """Small clustered images (near-duplicates exist, so stage 2 has something to do)."""
    rng = np.random.default_rng(seed)
    imgs = []
    for c in counts:
        k = max(2, c // 12)
        centres = rng.standard_normal((k, d))
        centres /= np.linalg.norm(centres, axis=1, keepdims=True)
        x = centres[rng.integers(0, k, size=c)] + rng.standard_normal((c, d)) * (0.2 / np.sqrt(d))
        x *= rng.lognormal(0, 0.3, size=(c, 1))
        imgs.append(x.astype(np.float32))
    dens = rng.uniform(0.1, 0.9, len(counts)).astype(np.float32)
    p = dict(synth.DEFAULT_PARAMS, iters=30)
    p.update(params)
    return synth.pack(0, dtype, imgs, dens, p)


@pytest.mark.parametrize("override", [
    dict(ratio=0.9),                     # tall and narrow: more kept tokens than a workgroup's registers hold
    dict(ratio=0.9, iters=0),
    dict(ratio=0.9, iters=1),
    dict(ratio=0.995),                   # a handful of pruned tokens per image (fewer than eight columns)
    dict(ratio=0.6, eps=1.0),            # wide pruned sets, the literal Appendix C
    dict(ratio=0.6, eps=0.02),           # exp range beyond fp32: the kernel matrix stays fp64
    dict(ratio=0.6, z=1.0),
    dict(ratio=0.45, alpha=0.5),         # more pruned than kept
])
def test_multi_workgroup_sinkhorn_variants(override):
    """Images beyond the register-resident shapes (600-900 tokens), bf16 width 1024."""
    batch = _clustered([600, 777, 900, 64, 513], 1024, "bf16", 21, **override)
    f = hz.run_prune(batch)
    rep = hz.compare_batch(batch, f, staged=False)
    _log(rep, f"sweep {override}")
    s = hz.run_staged(batch)
    rep2 = hz.compare_batch(batch, s, staged=True)
    rows = int(s["out_offsets"][-1])
    np.testing.assert_array_equal(f["out"][:rows], s["out"][:rows])
    np.testing.assert_array_equal(f["pair"], s["pair"])


@pytest.mark.parametrize("share", ["0", "5", "16"])
def test_streaming_kernels_with_a_share_of_streaming_loads(monkeypatch, share):
    """The streaming Sinkhorn kernels read the part of their matrices that the memory-side cache
    cannot keep with streaming loads.  The share is worked out from the matrices' size on the
    device; here it is fixed from the host (none, some, all of every 16 strips), on images wide
    and narrow enough for both load paths of the row kernel: the same bits each time, and right."""
    batch = _clustered([1800, 1500, 700, 2400], 256, "bf16", 41, ratio=0.45, iters=9)
    monkeypatch.delenv("RTPRUNE_SWEEP_STREAM_16THS", raising=False)
    ref = hz.run_prune(batch)
    assert ref["rc"] == 0 and ref["status"] == 0
    monkeypatch.setenv("RTPRUNE_SWEEP_STREAM_16THS", share)
    f = hz.run_prune(batch)
    assert f["rc"] == 0 and f["status"] == 0
    np.testing.assert_array_equal(ref["out"], f["out"])
    np.testing.assert_array_equal(ref["pair"], f["pair"])
    if share == "5":
        _log(hz.compare_batch(batch, f, images=[2, 3]), "sweep, 5/16 streamed")


@pytest.mark.parametrize("copies", [1, 12])
@pytest.mark.parametrize("D", [128, 384, 1152])
def test_tiled_merge_at_the_edges_of_its_tiles(D, copies):
    """Tiles of 128 kept rows x 128 (small batches) or 256 features (others; a width that is an odd multiple of 128
    leaves half of the last one), 32 pruned rows a step: row counts around the tile's, pruned counts around a step's."""
    shapes = [(1, 65), (63, 96), (64, 97), (65, 127), (127, 128), (128, 129), (129, 66), (255, 95), (257, 160)] * copies
    batch = _clustered([m + r for m, r in shapes], D, "bf16", 45, iters=12, ratio=0.55)
    keep = [m for m, _ in shapes]
    s = hz.run_staged(batch, keep_counts_in=keep)
    assert s["status"] == 0
    rep = hz.compare_batch(batch, s, staged=True, keep_counts=keep, images=list(range(9)) + [len(shapes) - 1])
    _log(rep, f"tiled merge {D} {copies}")


@pytest.mark.parametrize("copies", [1, 40])
@pytest.mark.parametrize("D", [128, 384, 640, 1152])
def test_tiled_merge_over_its_list(D, copies):
    """Pruned sets of 65 to 127 tokens under a fixed retention are merged over the list of them, in narrow tiles when they
    are few (4 images on the list) or the width leaves much of a wide one unused, else in wide ones (160 images of four rows
    of three or five tiles); short pages that are not on it lie between them."""
    counts = [400, 90, 331, 508, 200, 330] * copies
    batch = _clustered(counts, D, "bf16", 46, iters=9, ratio=0.7504)
    assert batch.max_tokens == 508
    f = hz.run_prune(batch)
    assert f["rc"] == 0 and f["status"] == 0
    pruned = np.diff(batch.offsets) - f["keep"]
    assert pruned.max() < 128 and (pruned > 64).sum() == 4 * copies and pruned.min() <= 64
    rep = hz.compare_batch(batch, f, images=list(range(6)) + [len(counts) - 3, len(counts) - 1])
    _log(rep, f"tiled merge list {D} {copies}")


def test_tall_register_shapes_at_their_edges():
    """Kept and pruned counts on both sides of the limits of the two shapes that hold
    a tall image (more than 512 rows) in one workgroup's registers: 1535 x 15
    (eight waves, all columns per lane) and 1216 x 64 (fp32-held matrix)."""
    shapes = [(1216, 64), (1217, 64), (1216, 65), (1535, 15), (1536, 15), (700, 16), (512, 1), (1535, 16),
              (600, 33), (1000, 1)]
    batch = _clustered([m + r for m, r in shapes], 128, "bf16", 24, iters=40)
    keep = [m for m, _ in shapes]
    s = hz.run_staged(batch, keep_counts_in=keep)
    rep = hz.compare_batch(batch, s, staged=True, keep_counts=keep)
    _log(rep, "tall shapes")
    assert rep.max_score_abs <= hz.SCORE_ATOL


def test_scores_of_more_workgroups_than_one_launch_takes():
    """fp32 tokens, 16 384 images of which one is long: 18.5 million workgroups of the score pass,
    where a launch takes fewer than 2^24 of 256 threads.  Images on both sides of where the second
    launch begins."""
    counts = [3] * 16383 + [4512]
    batch = _clustered(counts, 8, "f32", 61, dynamic=1, ratio_min=0.6, iters=3)
    f = hz.run_prune(batch)
    assert f["rc"] == 0 and f["status"] == 0
    assert (np.diff(batch.offsets) - f["keep"])[:-1].max() > 0
    first = ((1 << 24) - 2) // (282 * 4)                         # images of the first launch
    rep = hz.compare_batch(batch, f, images=[0, 1, 2, 5000] + list(range(first - 40, first + 40)) + [16382, 16383])
    _log(rep, "two launches of the score pass")


@pytest.mark.parametrize("override", [dict(), dict(iters=0), dict(iters=1), dict(iters=7), dict(eps=0.02),
                                      dict(eps=1.0, z=1.0, alpha=0.4)])
def test_multi_workgroup_resident_sinkhorn_at_its_edges(override):
    """At most 128 pruned tokens and more rows than the one-workgroup shapes of a large-image batch
    take: the kernel that keeps the matrix on chip
    across a cluster of workgroups (224 rows each while eight cover the image, else 448), on both
    sides of its limits and of its row strips; with eps = 0.02 exp's range does not fit fp32 and the streaming kernels take
    them all.  An odd and an even iteration count (the exchange buffers alternate)."""
    shapes = [(513, 100), (896, 128), (897, 128), (896, 129), (1300, 40), (600, 65), (1217, 64), (1216, 64),
              (449, 127), (3584, 128), (3585, 100), (2000, 17), (1792, 128), (1793, 100), (673, 90), (672, 128)]
    batch = _clustered([m + r for m, r in shapes], 128, "bf16", 35, **dict(dict(iters=40), **override))
    keep = [m for m, _ in shapes]
    s = hz.run_staged(batch, keep_counts_in=keep)
    assert s["status"] == 0
    rep = hz.compare_batch(batch, s, staged=True, keep_counts=keep)
    _log(rep, f"cluster shapes {override}")
    assert rep.max_score_abs <= hz.SCORE_ATOL


@pytest.mark.parametrize("override", [dict(), dict(iters=0), dict(iters=1), dict(iters=8)])
def test_multi_workgroup_resident_sinkhorn_wide_strips_at_their_edges(override):
    """More than 128 pruned tokens: the same kernel with strips of 144 rows x 576 columns (up to
    eight workgroups, 1152 rows), on both sides of its limits and of its strips; what lies beyond
    goes to the streaming kernels."""
    shapes = [(560, 523), (144, 576), (145, 129), (288, 300), (289, 300), (1152, 576), (1153, 576), (1152, 577),
              (1008, 129), (700, 200), (513, 130)]
    batch = _clustered([m + r for m, r in shapes], 128, "bf16", 38, **dict(dict(iters=31), **override))
    keep = [m for m, _ in shapes]
    s = hz.run_staged(batch, keep_counts_in=keep)
    assert s["status"] == 0
    rep = hz.compare_batch(batch, s, staged=True, keep_counts=keep)
    _log(rep, f"cluster wide strips {override}")
    assert rep.max_score_abs <= hz.SCORE_ATOL


@pytest.mark.parametrize("override", [dict(), dict(iters=0), dict(iters=1), dict(iters=6)])
def test_multi_workgroup_resident_sinkhorn_widest_strips_at_their_edges(override):
    """More than 576 pruned tokens (or more than 1152 kept rows with more than 128): strips of 80
    rows x 960 columns, up to sixteen workgroups.  Under the retention of these parameters the
    longest image fits, so a slot has sixteen workgroups; what lies beyond the shape goes to the
    one-workgroup general kernel."""
    shapes = [(1238, 899), (1280, 960), (80, 960), (81, 577), (1153, 300), (1280, 129), (640, 700), (1200, 961),
              (1281, 600), (560, 523), (700, 100)]
    batch = _clustered([m + r for m, r in shapes], 128, "bf16", 40, **dict(dict(iters=17, ratio=1280.0 / 2240.0), **override))
    assert batch.max_tokens == 2240                      # 1280 + 960: the retention keeps 1280 of them
    keep = [m for m, _ in shapes]
    s = hz.run_staged(batch, keep_counts_in=keep)
    assert s["status"] == 0
    rep = hz.compare_batch(batch, s, staged=True, keep_counts=keep)
    _log(rep, f"cluster widest strips {override}")
    assert rep.max_score_abs <= hz.SCORE_ATOL


@pytest.mark.parametrize("top,shapes,iters", [
    # strips of 64 rows x 1408 columns, 24 to a slot (more than an XCD's half: consecutive workgroups)
    ((1500, 1400), [(64, 1408), (65, 1408), (1492, 1408), (40, 1000), (2, 1200), (700, 961), (300, 130), (900, 128)], 7),
    # strips of 48 rows x 1792 columns, 27 to a slot; 1793 columns are the general kernel's
    ((1250, 1750), [(48, 1792), (49, 1792), (1208, 1792), (1200, 129), (97, 300), (60, 1793)], 6),
    ((1250, 1750), [(48, 1792), (433, 1409)], 0),
    # a few images: thin strips, 64 rows x 576 columns to a compute unit, up to sixteen workgroups
    ((1000, 287), [], 9),
    ((1024, 287), [(1, 200), (64, 576), (65, 576)], 9),
    ((420, 280), [(129, 300)], 1),
])
def test_multi_workgroup_strips_at_their_edges(top, shapes, iters):
    """The strip shapes beyond the first two and the thin strips of small batches, on both sides of
    their limits: the longest image and the retention choose the shape of the launch."""
    shapes = [top] + shapes
    batch = _clustered([m + r for m, r in shapes], 64, "f32", 43, iters=iters, ratio=top[0] / (top[0] + top[1]))
    assert batch.max_tokens == sum(top)
    keep = [m for m, _ in shapes]
    s = hz.run_staged(batch, keep_counts_in=keep)
    assert s["status"] == 0
    rep = hz.compare_batch(batch, s, staged=True, keep_counts=keep)
    _log(rep, f"strips {top}")


@pytest.mark.parametrize("params,shapes,streams", [
    # the parameters expect 341 pruned of 2137: two strip shapes and the streaming kernels in one call
    (dict(ratio=0.84), [(1238, 899), (1796, 341), (560, 523), (145, 129), (81, 577), (80, 960), (300, 1100), (700, 100)], True),
    # they expect clusters of up to 224 x 128 rows: strips all the same, nothing streamed
    (dict(ratio=0.9), [(560, 523), (720, 363), (400, 683), (513, 130), (144, 577), (975, 108)], False),
    (dict(dynamic=1, ratio_min=0.9), [(560, 523), (950, 133), (400, 683), (975, 108)], False),
])
def test_kept_counts_of_the_callers_own_in_several_strip_shapes(params, shapes, streams):
    """Staged calls whose kept counts have nothing to do with the parameters: the strips take them by their
    sizes, in slots as large as the images need, several images to a slot."""
    shapes = shapes + [(m - 1 - k, r - k) for k in range(3) for m, r in shapes[1:]]
    batch = _clustered([m + r for m, r in shapes], 64, "f32", 62, iters=7, **params)
    keep = [m for m, _ in shapes]
    rt.rtprune_profile_only(None)
    rt.rtprune_profile_enable(1)
    s = hz.run_staged(batch, keep_counts_in=keep)
    rc, prof = rt.rtprune_profile_summary()
    rt.rtprune_profile_enable(0)
    assert s["status"] == 0 and rc == 0
    launches = {r["kernel"]: r["launches"] for r in prof}
    assert "k_sinkhorn_strips" in launches
    to = rt.rtprune_sinkhorn_routes(len(shapes), batch.max_tokens, rt.make_params(batch.params), 1, keep, [r for _, r in shapes])[1]
    assert (to[:3] & 15 == rt.RTP_ROUTE_STRIPS).all() and streams == bool((to & 15 == rt.RTP_ROUTE_STREAMED).any()), to
    _log(hz.compare_batch(batch, s, staged=True, keep_counts=keep), f"own counts {params}")


def test_dynamic_retention_in_two_strip_shapes_through_the_fused_call():
    """A clamp that allows more than 576 pruned tokens: pages of up to 576 pruned tokens in one strip shape, the
    longest in the other, several images to a slot; fused = staged bit for bit."""
    rng = np.random.default_rng(63)
    counts = [int(c) for c in rng.integers(700, 1080, size=44)] + [1450, 1500]
    batch = _clustered(counts, 64, "f32", 63, dynamic=1, ratio_min=0.55, phi_lo=0.0, phi_hi=1e-3, iters=6)
    batch.density[-2:] = 0.0                                     # (these two at the clamp)
    rt.rtprune_profile_only(None)
    rt.rtprune_profile_enable(1)
    f = hz.run_prune(batch)
    rc, prof = rt.rtprune_profile_summary()
    rt.rtprune_profile_enable(0)
    assert f["rc"] == 0 and f["status"] == 0 and rc == 0
    pruned = np.diff(batch.offsets) - f["keep"]
    assert ((pruned > 128) & (pruned <= 576)).sum() > 32 and (pruned > 576).any(), pruned
    ms = {r["kernel"]: r["total_ms"] for r in prof}
    assert "k_sinkhorn_strips" in ms, ms
    rep = hz.compare_batch(batch, f, images=list(range(0, 46, 5)) + [45])
    _log(rep, "dynamic, two strip shapes")
    s = hz.run_staged(batch)
    _assert_fused_equals_staged(f, s, batch)


# Images at the edges of the strips' forms, by strip shape: what the retention expects of the longest page (which
# chooses the shape), and (kept, pruned): (workgroups, whether everybody reads everybody's sums in one trip).
# tests/test_strip_forms_cpu.py asks the kernels' own rules for the same.
STRIP_EDGES = {
    "72 x 576": ((788, 570), {
        (72, 300): (1, True), (73, 576): (2, True), (144, 575): (2, True), (145, 576): (3, True), (288, 576): (4, True),
        (289, 463): (5, True), (289, 464): (5, False), (360, 573): (5, False), (576, 289): (8, True), (576, 290): (8, False),
        (577, 574): (9, False), (788, 570): (11, False), (860, 190): (12, True), (860, 192): (12, False)}),
    "40 x 960": ((776, 582), {
        (40, 900): (1, True), (41, 577): (2, True), (80, 960): (2, True), (81, 301): (3, True), (120, 770): (3, True),
        (120, 772): (3, False), (160, 579): (4, True), (160, 580): (4, False), (200, 463): (5, True), (201, 957): (6, False),
        (640, 143): (16, True), (640, 144): (16, False), (680, 134): (17, True), (776, 582): (20, False)}),
}


@pytest.mark.parametrize("iters", [1, 2, 3, 6])
@pytest.mark.parametrize("shape", list(STRIP_EDGES))
def test_strips_of_half_a_compute_unit_at_their_edges(shape, iters):
    """Workgroups of 72 x 576 and 40 x 960: one of them, the most that everybody reads everybody's sums of
    (2320) and the first that deal the columns out, and pruned counts whose shares and pairs end unevenly."""
    top, forms = STRIP_EDGES[shape]
    shapes = list(forms) * 2                           # (more images than thin strips are for)
    batch = _clustered([m + r for m, r in shapes], 128, "bf16", 44, iters=iters, ratio=top[0] / (top[0] + top[1]))
    assert batch.max_tokens == sum(top)
    keep = [m for m, _ in shapes]
    s = hz.run_staged(batch, keep_counts_in=keep)
    assert s["status"] == 0
    rep = hz.compare_batch(batch, s, staged=True, keep_counts=keep, images=list(range(len(forms))))
    _log(rep, f"half strips {shape} {iters}")


def test_multi_workgroup_resident_sinkhorn_wide_strips_fill_the_chip():
    """A fixed retention under which the longest image takes four strips: slots of four workgroups,
    64 of them, more images than slots, through the fused call (no launches of the streaming
    kernels: the profile says which kernels ran); fused = staged bit for bit."""
    rng = np.random.default_rng(39)
    counts = [int(c) for c in rng.integers(700, 1084, size=70)] + [1083]
    batch = _clustered(counts, 256, "bf16", 39, ratio=560.0 / 1083.0, iters=12)
    rt.rtprune_profile_only(None)
    rt.rtprune_profile_enable(1)
    f = hz.run_prune(batch)
    rc, prof = rt.rtprune_profile_summary()
    rt.rtprune_profile_enable(0)
    assert f["rc"] == 0 and f["status"] == 0 and rc == 0
    ms = {r["kernel"]: r["total_ms"] for r in prof}
    # (the streaming kernels' 2 T + 3 launches are recorded under k_sinkhorn, with the general
    # kernel's one: far more than the 0.1 ms allowed here if they were issued)
    assert "k_sinkhorn_strips" in ms and ms.get("k_sinkhorn", 0.0) < 0.1, ms
    rc, to = rt.rtprune_sinkhorn_routes(len(counts), batch.max_tokens, rt.make_params(batch.params), 0, f["keep"],
                                        np.diff(batch.offsets) - f["keep"])
    assert rc == 0 and (to & 15 == rt.RTP_ROUTE_STRIPS).all()
    rep = hz.compare_batch(batch, f, images=list(range(0, 71, 6)) + [70])
    _log(rep, "cluster wide strips, fused, 71 images")
    s = hz.run_staged(batch)
    rows = int(s["out_offsets"][-1])
    np.testing.assert_array_equal(f["out"][:rows], s["out"][:rows])
    np.testing.assert_array_equal(f["pair"], s["pair"])
    for _ in range(3):                                           # run-to-run determinism of the exchange
        g = hz.run_prune(batch)
        np.testing.assert_array_equal(f["out"], g["out"])
        np.testing.assert_array_equal(f["pair"], g["pair"])


def test_multi_workgroup_resident_sinkhorn_through_the_fused_call_many_images():
    """More such images than the launch has cluster slots (each slot takes several in turn), of
    different heights, through the fused call; fused = staged bit for bit."""
    rng = np.random.default_rng(36)
    counts = [int(c) for c in rng.integers(620, 1500, size=40)]
    batch = _clustered(counts, 1024, "bf16", 36, ratio=0.93, iters=21)
    f = hz.run_prune(batch)
    assert f["rc"] == 0 and f["status"] == 0
    pruned = np.diff(batch.offsets) - f["keep"]
    assert (pruned > 16).all() and (pruned <= 128).all() and (f["keep"] > 512).all()
    rep = hz.compare_batch(batch, f, images=range(0, 40, 3))
    _log(rep, "cluster fused, 40 images")
    s = hz.run_staged(batch)
    rows = int(s["out_offsets"][-1])
    np.testing.assert_array_equal(f["out"][:rows], s["out"][:rows])
    np.testing.assert_array_equal(f["pair"], s["pair"])
    g = hz.run_prune(batch)                                      # run-to-run determinism
    np.testing.assert_array_equal(f["out"], g["out"])


def test_multi_workgroup_sinkhorn_gives_up_instead_of_waiting_for_ever(monkeypatch):
    """The cluster kernel's waits are bounded.  With no poll allowed (the host-side test switch) the first meeting
    gives up: the call returns, every kernel ends, and the status word says that the wait timed out.  With a single
    poll a workgroup that does not find its cluster complete at once gives up.  (One run of many found them in
    step at every meeting: an arrival takes longer to reach the counter than three workgroups started
    together are apart.)  Then the call is right to the last bit.  The next call, with the usual bound, is right again."""
    batch = _clustered([700, 900, 1200, 650], 1024, "bf16", 37, ratio=0.93, iters=30)
    ref = hz.run_prune(batch)
    assert ref["rc"] == 0 and ref["status"] == 0
    _log(hz.compare_batch(batch, ref), "before a timed-out call")
    for polls in (0, 1):
        monkeypatch.setenv("RTPRUNE_SYNC_SPIN_LIMIT", str(polls))
        f = hz.run_prune(batch)
        assert f["rc"] == 0
        assert f["status"] & rt.RTP_DEV_SYNC_TIMEOUT or (polls and f["status"] == 0), f["status"]
        if f["status"] == 0:
            np.testing.assert_array_equal(f["out"], ref["out"])
            np.testing.assert_array_equal(f["pair"], ref["pair"])
        monkeypatch.delenv("RTPRUNE_SYNC_SPIN_LIMIT")
        g = hz.run_prune(batch)
        assert g["rc"] == 0 and g["status"] == 0
        np.testing.assert_array_equal(g["out"], ref["out"])
        np.testing.assert_array_equal(g["pair"], ref["pair"])


# batches whose images go through the strips: (sizes, retention, iterations, whether their exchange takes one trip:
# tests/test_strip_forms_cpu.py).  Several images to a slot of 3, 4, 16 and, across the XCDs, 24 compute units; thin
# strips of one page.
STRIP_BATCHES = {
    "3 units, one trip": ([700] * 3 + list(range(520, 700)), 560.0 / 1083.0, 5, True),
    "4 units": ([1083] * 3 + list(range(800, 1070)), 560.0 / 1083.0, 5, False),
    "16 units": ([2137] + list(range(1700, 1900, 11)), 1238.0 / 2137.0, 5, False),
    "24 units": ([2900] + list(range(2860, 2895, 2)), 1500.0 / 2900.0, 4, False),
    "one page": ([1156], 0.75, 9, False),
    "one page, one trip": ([560], 0.75, 9, True),
}


@pytest.mark.parametrize("name", list(STRIP_BATCHES))
def test_strip_slots_that_do_not_get_complete_leave_their_images_to_the_next_launch(monkeypatch, name):
    """A strip slot whose workgroups are not all resident in time is given up, and a launch of whole compute units does
    its images.  With the host-side test switch every slot is given up, or those that a few polls do not find complete:
    same bits as with none, and right."""
    counts, ratio, iters, _ = STRIP_BATCHES[name]
    batch = _clustered(counts, 16, "f32", 64, ratio=ratio, iters=iters)
    f = hz.run_prune(batch)
    assert f["rc"] == 0 and f["status"] == 0
    m, r = f["keep"], np.diff(batch.offsets) - f["keep"]
    rc, to = rt.rtprune_sinkhorn_routes(len(counts), batch.max_tokens, rt.make_params(batch.params), 0, m, r)
    assert rc == 0 and (to & 15 == rt.RTP_ROUTE_STRIPS).all()
    _log(hz.compare_batch(batch, f, images=sorted({0, 1 % len(counts), len(counts) // 2, len(counts) - 1})), name)
    for polls in (0, 1, 4, 16):
        monkeypatch.setenv("RTPRUNE_STRIP_FORM_POLLS", str(polls))
        g = hz.run_prune(batch)
        assert g["rc"] == 0 and g["status"] == 0
        for k in ("out", "pair", "sel", "keep"):
            np.testing.assert_array_equal(f[k], g[k])


@pytest.mark.parametrize("iters", [0, 1, 4])
@pytest.mark.parametrize("top,shapes", [
    ((788, 570), [(72, 300), (73, 576), (145, 200), (360, 463), (360, 464), (576, 289), (577, 290), (217, 575)]),
    ((776, 582), [(40, 900), (41, 577), (81, 300), (160, 578), (161, 579), (401, 957), (800, 558)]),
    ((1500, 1400), [(32, 1408), (33, 1408), (65, 1200), (1492, 1400)]),
    ((1250, 1750), [(24, 1792), (25, 1700), (49, 1792), (1208, 1792)]),
])
def test_slots_given_up_on_workgroups_of_two_teams(monkeypatch, top, shapes, iters):
    """The launch behind the strips does two of their workgroups' parts in each of its own: images of one part
    (the other half of the workgroup is there for the barriers), of an even and of an odd number, several to a slot,
    both forms of the exchange, every strip shape.  Same bits as the strips'."""
    shapes = [top] + shapes * 2
    batch = _clustered([m + r for m, r in shapes], 16, "f32", 66, iters=iters, ratio=top[0] / (top[0] + top[1]))
    keep = [m for m, _ in shapes]
    f = hz.run_staged(batch, keep_counts_in=keep)
    assert f["status"] == 0
    _log(hz.compare_batch(batch, f, staged=True, keep_counts=keep, images=list(range(len(shapes) // 2 + 1))), f"two teams {top}")
    monkeypatch.setenv("RTPRUNE_STRIP_FORM_POLLS", "0")
    g = hz.run_staged(batch, keep_counts_in=keep)
    assert g["status"] == 0
    for k in ("out", "pair", "plan"):
        np.testing.assert_array_equal(f[k], g[k])


@pytest.mark.parametrize("names,wide", [
    (("16 units",) * 4, False),
    (("16 units", "24 units", "4 units", "24 units"), False),
    (("3 units, one trip", "16 units", "3 units, one trip", "24 units"), False),
    (("16 units", "4 units", "3 units, one trip", "16 units"), True),
])
def test_strip_calls_on_four_streams_at_once(names, wide):
    """Four calls at a time, a stream each, whose slots compete for the compute units: all end without a time-out
    and with the bits of a call alone.  `wide`: bf16 tokens of 640 features, whose tiled kernels, of other register counts,
    run beside the strips."""
    jobs = []
    for i, name in enumerate(names):
        counts, ratio, iters, _ = STRIP_BATCHES[name]
        if wide:
            counts = counts[:60]
        batch = _clustered(counts, 640 if wide else 16, "bf16" if wide else "f32", 70 + i, ratio=ratio, iters=40)
        ref = hz.run_prune(batch)
        assert ref["rc"] == 0 and ref["status"] == 0
        db, p = rt.upload(batch), rt.make_params(batch.params)
        ws = rt.alloc_workspace(db)
        out = torch.zeros_like(db.tokens)
        off = torch.zeros(db.B + 1, dtype=torch.int32, device="cuda:0")
        pair = torch.zeros(db.total_tokens, dtype=torch.int32, device="cuda:0")
        jobs.append((ref, db, p, ws, out, off, pair, torch.cuda.Stream()))
    torch.cuda.synchronize()
    for _ in range(5):
        for ref, db, p, ws, out, off, pair, stream in jobs:
            assert rt.rtprune_prune(db, None, p, out, off, None, None, pair, None, ws, stream=stream) == rt.RTP_OK
    torch.cuda.synchronize()
    for ref, db, p, ws, out, off, pair, stream in jobs:
        assert hz.device_status(ws) == 0
        rows = int(ref["out_offsets"][-1])
        np.testing.assert_array_equal(hz._np(out)[:rows], ref["out"][:rows])
        np.testing.assert_array_equal(pair.cpu().numpy(), ref["pair"])


@pytest.mark.parametrize("name", list(STRIP_BATCHES))
def test_strips_give_up_instead_of_waiting_for_ever(monkeypatch, name):
    """The strips' own waits are bounded, in both forms of their exchange.  With no poll allowed the first meeting
    gives up; with a few, workgroups in step may get through it and through some iterations: the call either says
    that a wait timed out or is right to the last bit."""
    counts, ratio, iters, _ = STRIP_BATCHES[name]
    batch = _clustered(counts[:6], 16, "f32", 65, ratio=ratio, iters=iters)
    ref = hz.run_prune(batch)
    assert ref["rc"] == 0 and ref["status"] == 0
    _log(hz.compare_batch(batch, ref, images=[0]), name)
    for polls in (0, 1, 2, 5):
        monkeypatch.setenv("RTPRUNE_SYNC_SPIN_LIMIT", str(polls))
        f = hz.run_prune(batch)
        assert f["rc"] == 0 and f["status"] in ((0, rt.RTP_DEV_SYNC_TIMEOUT) if polls else (rt.RTP_DEV_SYNC_TIMEOUT,))
        if f["status"] == 0:
            np.testing.assert_array_equal(f["out"], ref["out"])
        print(f"[{name}] {polls} polls: status {f['status']}", flush=True)
        monkeypatch.delenv("RTPRUNE_SYNC_SPIN_LIMIT")
        g = hz.run_prune(batch)
        assert g["rc"] == 0 and g["status"] == 0
        np.testing.assert_array_equal(g["out"], ref["out"])
        np.testing.assert_array_equal(g["pair"], ref["pair"])


@pytest.mark.parametrize("override", [dict(), dict(eps=0.02), dict(iters=0), dict(iters=1)])
def test_wide_register_shapes_at_their_edges(override):
    """Images of at most 512 tokens with 65 to 225 pruned ones, on both sides of the
    limits of the three shapes that hold such a matrix as fp32 in one workgroup's
    registers (448 x 128, 384 x 192, 320 x 224); with eps = 0.02 exp's range does not
    fit fp32 and the general kernel takes them all."""
    shapes = [(447, 65), (384, 128), (385, 127), (383, 129), (320, 192), (321, 191), (288, 224), (287, 225),
              (100, 200), (240, 160), (64, 65)]
    batch = _clustered([m + r for m, r in shapes], 128, "bf16", 27, **dict(dict(iters=40), **override))
    assert max(m + r for m, r in shapes) <= 512
    keep = [m for m, _ in shapes]
    s = hz.run_staged(batch, keep_counts_in=keep)
    rep = hz.compare_batch(batch, s, staged=True, keep_counts=keep)
    _log(rep, f"wide shapes {override}")
    assert rep.max_score_abs <= hz.SCORE_ATOL


@pytest.mark.parametrize("override", [dict(), dict(eps=0.02), dict(iters=0), dict(iters=1), dict(eps=1.0, iters=100)])
def test_64_column_register_shapes_at_their_edges(override):
    """41 to 64 pruned tokens: the 384 x 64 shape that holds the matrix as fp32 (two workgroups
    per compute unit) on both sides of its limits, and the 512 x 64 fp64 shape beyond them; with
    eps = 0.02 exp's range does not fit fp32 and the fp64 shape takes them all."""
    shapes = [(384, 64), (385, 64), (384, 41), (383, 63), (337, 63), (447, 64), (50, 49), (1, 64), (448, 41)]
    batch = _clustered([m + r for m, r in shapes], 128, "bf16", 33, **dict(dict(iters=40), **override))
    keep = [m for m, _ in shapes]
    s = hz.run_staged(batch, keep_counts_in=keep)
    rep = hz.compare_batch(batch, s, staged=True, keep_counts=keep)
    _log(rep, f"64-column shapes {override}")
    assert rep.max_score_abs <= hz.SCORE_ATOL


# kept x pruned at the limits of the images that one wave and two waves take (the dustbins are one more row and column), rows
# past which a wave's share of them ends among them; neighbours take different numbers of waves
SHORT_EDGES = [(127, 15), (128, 15), (63, 8), (255, 8), (64, 7), (127, 8), (400, 15), (64, 15), (256, 15), (63, 15), (497, 15),
               (447, 7), (448, 7), (128, 8), (1, 15), (192, 9), (126, 15), (503, 8), (255, 15), (128, 7), (320, 7), (383, 7), (384, 7),
               (2, 8), (30, 2)]


@pytest.mark.parametrize("copies", [1, 24])
@pytest.mark.parametrize("override", [dict(iters=0), dict(iters=1), dict(iters=3), dict(iters=60)])
def test_one_and_two_wave_images_at_their_edges(override, copies):
    """Up to 15 pruned tokens against the oracle, with a SIMD to a wave and with eight waves to a workgroup."""
    keep = [m for m, _ in SHORT_EDGES] * copies
    batch = _clustered([m + r for m, r in SHORT_EDGES], 128, "f32", 55, **override)
    many = synth.subset(batch, list(range(len(SHORT_EDGES))) * copies)
    g = hz.run_staged(many, keep_counts_in=keep)
    rep = hz.compare_batch(batch, dict(g, out_offsets=g["out_offsets"][:len(SHORT_EDGES) + 1],
                                       plan_offsets=g["plan_offsets"][:len(SHORT_EDGES) + 1]),
                           staged=True, keep_counts=keep[:len(SHORT_EDGES)])
    _log(rep, f"one and two waves {override} x{copies}")
    for key, size in (("out", sum(m for m, _ in SHORT_EDGES)), ("pair", sum(m + r for m, r in SHORT_EDGES)),
                      ("plan", sum(m * r for m, r in SHORT_EDGES))):
        for c in range(1, copies):
            np.testing.assert_array_equal(g[key][c * size:(c + 1) * size], g[key][:size])


def test_one_and_two_wave_images_run_side_by_side():
    """Images of one wave, which meet no barrier, beside images of two, which meet one an iteration: no workgroup holds
    both, or the latter would not start before the former have ended.  (These parameters move for 2500 iterations.)"""
    params = dict(iters=2500, z=1.0, eps=0.0034)
    def ms(shapes):
        batch = _clustered([m + r for m, r in shapes], 128, "f32", 57, **params)
        times = []
        for _ in range(3):
            rt.rtprune_profile_enable(1)
            hz.run_staged(batch, keep_counts_in=[m for m, _ in shapes])
            rc, prof = rt.rtprune_profile_summary()
            rt.rtprune_profile_enable(0)
            assert rc == rt.RTP_OK
            times.append(next(k["total_ms"] for k in prof if k["kernel"] == "k_sinkhorn_regs"))
        return min(times)
    one, two, both = ms([(100, 15)] * 40), ms([(300, 15)] * 40), ms([(100, 15), (300, 15)] * 40)
    print(f"\none wave {one:.3f} ms, two waves {two:.3f} ms, both {both:.3f} ms", flush=True)
    assert one > 0.2 and two > 0.2                       # (not settled after a few)
    assert both < max(one, two) + 0.5 * min(one, two)


# kept x pruned around the batches of 128 rows (the dustbin row is one more), the 32, 48 and 64 columns and the 352
# rows that four waves hold
GRID_EDGES = [(1, 16), (31, 31), (126, 16), (127, 31), (128, 32), (129, 47), (254, 17), (255, 48), (256, 63), (257, 40),
              (351, 63), (352, 63), (351, 64), (383, 33), (384, 48), (448, 63), (464, 47), (480, 31), (495, 16)]


@pytest.mark.parametrize("override", [dict(iters=0), dict(iters=1), dict(iters=2), dict(iters=60), dict(iters=30, eps=0.02)])
def test_register_shapes_of_up_to_64_columns_at_their_edges(override):
    """16 to 64 pruned tokens against the oracle, in as many images as the chip has compute units for and among
    more of them: the same bits."""
    counts = [m + r for m, r in GRID_EDGES]
    keep = [m for m, _ in GRID_EDGES]
    assert max(counts) == 512 - 1
    fill = 300
    batch = _clustered(counts + [2] * fill, 128, "f32", 51, **override)
    few = synth.subset(batch, range(len(counts)))
    s = hz.run_staged(few, keep_counts_in=keep)
    rep = hz.compare_batch(few, s, staged=True, keep_counts=keep)
    _log(rep, f"64 columns {override}")
    g = hz.run_staged(batch, keep_counts_in=keep + [2] * fill)
    rows, cells, tokens = sum(keep), sum(m * r for m, r in GRID_EDGES), sum(counts)
    np.testing.assert_array_equal(s["out"][:rows], g["out"][:rows])
    np.testing.assert_array_equal(s["pair"][:tokens], g["pair"][:tokens])
    np.testing.assert_array_equal(s["plan"][:cells], g["plan"][:cells])


@pytest.mark.parametrize("override", [dict(iters=0), dict(iters=1), dict(iters=2), dict(iters=60)])
def test_tall_shape_of_up_to_31_columns_at_its_edges(override):
    """16 to 32 pruned tokens around the batches of 512 rows (the dustbin row is one more) and the limits of the shape."""
    shapes = [(512, 16), (513, 31), (640, 30), (1022, 17), (1023, 31), (1024, 20), (1151, 16), (1216, 31), (1216, 32), (900, 32)]
    batch = _clustered([m + r for m, r in shapes], 128, "bf16", 53, **override)
    keep = [m for m, _ in shapes]
    s = hz.run_staged(batch, keep_counts_in=keep)
    rep = hz.compare_batch(batch, s, staged=True, keep_counts=keep)
    _log(rep, f"tall 31 columns {override}")


def test_heavily_pruned_400_token_pages_fused():
    """Dynamic retention at its clamp on 400-token pages whose tokens resemble each other:
    160 pruned tokens per page, through the fused call."""
    rng = np.random.default_rng(28)
    d, imgs = 1024, []
    for c in [400, 400, 380, 256, 512]:
        common = rng.standard_normal(d)
        common /= np.linalg.norm(common)
        x = common[None, :] + rng.standard_normal((c, d)) / np.sqrt(d)
        dup = rng.integers(0, c, size=c // 5)
        x[rng.permutation(c)[:c // 5]] = x[dup] + rng.standard_normal((c // 5, d)) * (0.05 / np.sqrt(d))
        x *= rng.lognormal(0, 0.3, size=(c, 1))
        imgs.append(x.astype(np.float32))
    dens = np.array([0.05, 0.3, 0.1, 0.2, 0.15], dtype=np.float32)
    batch = synth.pack(0, "bf16", imgs, dens, dict(synth.DEFAULT_PARAMS, dynamic=1, iters=30))
    f = hz.run_prune(batch)
    pruned = np.diff(batch.offsets) - f["keep"]
    assert (pruned > 64).all(), pruned
    rep = hz.compare_batch(batch, f, staged=False)
    _log(rep, f"wide fused pruned={list(pruned)}")
    s = hz.run_staged(batch)
    rows = int(s["out_offsets"][-1])
    np.testing.assert_array_equal(f["out"][:rows], s["out"][:rows])
    np.testing.assert_array_equal(f["pair"], s["pair"])


@pytest.mark.parametrize("override", [dict(ratio=0.96), dict(ratio=0.99), dict(ratio=0.96, iters=0),
                                      dict(ratio=0.96, eps=0.02)])
def test_tall_images_fused(override):
    """Tiled-page sized images with few pruned tokens through the fused call."""
    batch = _clustered([1156, 1000, 800, 1300, 520, 1500], 1024, "bf16", 25, **override)
    f = hz.run_prune(batch)
    rep = hz.compare_batch(batch, f, staged=False)
    _log(rep, f"tall fused {override}")
    s = hz.run_staged(batch)
    rows = int(s["out_offsets"][-1])
    np.testing.assert_array_equal(f["out"][:rows], s["out"][:rows])
    np.testing.assert_array_equal(f["pair"], s["pair"])


# (T = 0 goes with eps = 1: at eps = 0.05 the unnormalised exp(S / eps) of hundreds of
# look-alike tokens sums to 1e4 and more per row, where fp32 accumulation noise alone
# exceeds the absolute bar)
@pytest.mark.parametrize("override", [dict(), dict(iters=0, eps=1.0), dict(iters=1), dict(eps=1.0),
                                      dict(z=0.9, alpha=0.3)])
def test_dynamic_ratio_on_tiled_page_sizes_with_many_pruned_tokens(override):
    """Dynamic retention on images of 700-1150 tokens whose tokens resemble each other
    (phi near 0.5), so that hundreds are pruned: the retention clamp's bound is reached,
    and the sweep and tiled kernels serve a batch sized by that bound."""
    rng = np.random.default_rng(26)
    d, imgs = 1024, []
    for c in [800, 1150, 700, 1000, 300, 1156]:
        common = rng.standard_normal(d)
        common /= np.linalg.norm(common)
        x = common[None, :] + rng.standard_normal((c, d)) / np.sqrt(d)
        dup = rng.integers(0, c, size=c // 5)                  # near-copies: clear partners
        x[rng.permutation(c)[:c // 5]] = x[dup] + rng.standard_normal((c // 5, d)) * (0.05 / np.sqrt(d))
        x *= rng.lognormal(0, 0.3, size=(c, 1))
        imgs.append(x.astype(np.float32))
    dens = np.array([0.05, 0.1, 0.3, 0.6, 0.2, 0.9], dtype=np.float32)
    p = dict(synth.DEFAULT_PARAMS, dynamic=1, iters=30)
    p.update(override)
    batch = synth.pack(0, "bf16", imgs, dens, p)
    f = hz.run_prune(batch)
    pruned = np.diff(batch.offsets) - f["keep"]
    assert (pruned[:4] > 64).all() and pruned.max() > 256, pruned   # beyond every register shape
    rep = hz.compare_batch(batch, f, staged=False)
    _log(rep, f"clamped {override} pruned={list(pruned)}")


@pytest.mark.parametrize("dtype,d", [("f32", 64), ("bf16", 72), ("bf16", 256), ("f32", 1280)])
def test_multi_workgroup_sinkhorn_other_widths(dtype, d):
    """The same images through the general score and merge kernels (fp32 tokens, odd widths)."""
    batch = _clustered([640, 530], d, dtype, 22, ratio=0.7)
    f = hz.run_prune(batch)
    rep = hz.compare_batch(batch, f, staged=False)
    _log(rep, f"sweep {dtype} D={d}")


@pytest.mark.parametrize("counts,ratio", [([260], 0.25), ([200, 7 + 193], 0.0174), ([321, 450], 0.4),
                                          ([130], 0.5), ([72, 71], 0.09), ([400], 0.8375)])
def test_matrix_core_tiles_at_their_edges(counts, ratio):
    """Pruned sets just above the tiled kernels' threshold (65 pruned tokens; the second
    image of the fifth case has 64 and stays below it) and around 192, tiles cut by both
    edges."""
    batch = _clustered(counts, 1024, "bf16", 23, ratio=ratio, iters=10)
    s = hz.run_staged(batch)
    rep = hz.compare_batch(batch, s, staged=True)
    _log(rep, f"tiles {counts} {ratio}")
    assert rep.max_score_abs <= hz.SCORE_ATOL
    f = hz.run_prune(batch)
    rows = int(s["out_offsets"][-1])
    np.testing.assert_array_equal(f["out"][:rows], s["out"][:rows])


@pytest.mark.parametrize("d,ratio", [(1024, 0.85), (1152, 0.55), (1280, 0.7)])
def test_score_kernels_of_small_and_large_batches(d, ratio):
    """Up to half a 128-row tile per compute unit the scores come from 16-row workgroups with the
    contraction split over their waves (width / 64 steps over four waves: even and uneven shares),
    beyond that from the 128-row ones: both against the oracle, at kept and pruned counts around
    their 16-row tiles, and the same image alone and in the large batch gives the same rows."""
    counts = [17, 31, 33, 64, 95, 100, 129, 140]
    batch = _clustered(counts + [40 + i % 9 for i in range(260)], d, "bf16", 44, ratio=ratio, iters=9)
    f = hz.run_prune(batch)
    _log(hz.compare_batch(batch, f, images=range(0, 12)), f"scores of a large batch {d}")
    small = synth.subset(batch, range(len(counts)))
    g = hz.run_prune(small)
    _log(hz.compare_batch(small, g), f"scores of a small batch {d}")
    rows = int(g["out_offsets"][-1])
    np.testing.assert_array_equal(f["out"][:rows], g["out"][:rows])


@pytest.mark.parametrize("d", [128, 384, 512, 896])
def test_tiled_scores_at_other_step_counts(d):
    """The tiled score kernel walks the width 64 elements a step, with three staging buffers
    and two accumulator sets in turn (a pattern of six steps): 2, 6, 8 and 14 steps, tiles cut
    by both edges, the staged call (scores entry by entry) and the fused one."""
    batch = _clustered([300, 457, 131], d, "bf16", 43, ratio=0.4, iters=10)
    s = hz.run_staged(batch)
    rep = hz.compare_batch(batch, s, staged=True)
    _log(rep, f"tiled scores D={d}")
    assert rep.max_score_abs <= hz.SCORE_ATOL
    f = hz.run_prune(batch)
    rows = int(s["out_offsets"][-1])
    np.testing.assert_array_equal(f["out"][:rows], s["out"][:rows])
    np.testing.assert_array_equal(f["pair"], s["pair"])


@pytest.mark.parametrize("counts,ratio,d", [
    ([100, 116, 96], 0.83, 1024),      # 17, 19 and 16 pruned tokens: the last stays with the vector kernel
    ([160, 161], 0.8, 1280),           # 32 pruned tokens (one operand block), 128 and 129 kept rows
    ([193, 40], 0.665, 1024),          # 64 pruned tokens, rows cut by a tile; a 13-token pruned set beside it
    ([400, 400], 0.8425, 1280),        # the paper's average retention on a 400-token page
    ([97, 50], 0.34, 256),             # fewer kept rows than a wave takes, 64 and 33 pruned
    ([120, 300], 0.6, 192),            # width a multiple of 64 only; the second image is beyond the range
    ([120], 0.6, 96),                  # width no multiple of 64: the vector kernel
    ([160, 97], 0.8, 64),              # half a stage of features, one, three, four and five stages
    ([97, 193], 0.67, 128),
    ([130, 97], 0.7, 384),
    ([160, 97], 0.8, 512),
    ([130, 97], 0.7, 640),
    ([400, 230], 0.8425, 1088),        # the last of nine stages has half of its features
    ([160, 193], 0.8, 1152),
])
def test_unstaged_matrix_core_merge_at_its_edges(counts, ratio, d):
    """Pruned sets of 17 to 64 tokens (the merge kernel that feeds the matrix cores straight
    from memory), at both ends of the range, with kept rows cut by its 32- and 128-row blocks."""
    batch = _clustered(counts, d, "bf16", 29, ratio=ratio, iters=10)
    on = dict(batch.params, mid_merge_min_images=1)   # (by default a few pages do not run it)
    s = hz.run_staged(batch, on)
    f = hz.run_prune(batch, on)
    rep = hz.compare_batch(batch, s, staged=True)
    _log(rep, f"mid merge {counts} {ratio} D={d}")
    rows = int(s["out_offsets"][-1])
    np.testing.assert_array_equal(f["out"][:rows], s["out"][:rows])
    v = hz.run_prune(batch)                         # and the same images through the vector kernel
    rep = hz.compare_batch(batch, v, staged=False)
    _log(rep, f"mid merge, vector kernel {counts} {ratio} D={d}")


def test_middling_merge_of_any_number_of_pages():
    """Two pages past a multiple of eight take no longer than the next multiple (a workgroup per row tile of each)."""
    def ms(count):
        batch = synth.gen_batch(9, images=[b % 8 for b in range(count)])
        batch.params.update(iters=1, mid_merge_min_images=1)
        times = []
        for _ in range(5):
            rt.rtprune_profile_enable(1)
            hz.run_prune(batch)
            rc, prof = rt.rtprune_profile_summary()
            rt.rtprune_profile_enable(0)
            assert rc == rt.RTP_OK
            times.append(next(k["total_ms"] for k in prof if k["kernel"] == "k_merge"))
        return min(times)
    few, many = ms(10), ms(16)
    print(f"\nmerge of 10 pages {few * 1e3:.1f} us, of 16 {many * 1e3:.1f} us", flush=True)
    assert few < 1.15 * many


def test_merge_without_workspace():
    """The merge entry point without a workspace (vector kernel for every small pruned set)."""
    import torch
    batch = _clustered([160, 97, 300, 40], 1024, "bf16", 31, ratio=0.7, iters=10)
    s = hz.run_staged(batch)
    db = rt.upload(batch, "cuda:0")
    dev = lambda a, t: torch.from_numpy(np.ascontiguousarray(a)).to(t).cuda()
    out = torch.zeros((int(s["out_offsets"][-1]), db.D), dtype=db.tokens.dtype, device="cuda:0")
    rt.check(rt.rtprune_merge(db, dev(s["sel"], torch.int32), dev(s["keep"], torch.int32),
                              dev(s["out_offsets"], torch.int32), dev(s["plan"], torch.float32),
                              dev(s["plan_offsets"], torch.int64), rt.make_params(batch.params), out, None))
    torch.cuda.synchronize()
    got = dict(s, out=hz._np(out))
    rep = hz.compare_batch(batch, got, staged=True)
    _log(rep, "merge without workspace")


def _merge_alone(tokens, counts, keep, plan, **params):
    """rtprune_merge on bf16 bits with kept tokens before the pruned ones, the caller's counts and the caller's plan."""
    import torch
    batch = synth.pack(0, "bf16", tokens, np.zeros(len(counts), np.float32), dict(synth.DEFAULT_PARAMS, dynamic=0, **params))
    db = rt.upload(batch, "cuda:0")
    ws = rt.alloc_workspace(db)
    ws.fill_(0xFF)
    dev = lambda a, t: torch.from_numpy(np.ascontiguousarray(a)).to(t).cuda()
    out_off = np.concatenate([[0], np.cumsum(keep)])
    plan_off = np.concatenate([[0], np.cumsum([m * (n - m) for n, m in zip(counts, keep)])])
    out = torch.zeros((int(out_off[-1]), db.D), dtype=db.tokens.dtype, device="cuda:0")
    rt.check(rt.rtprune_merge(db, dev(np.concatenate([np.arange(n) for n in counts]), torch.int32), dev(keep, torch.int32),
                              dev(out_off, torch.int32), dev(plan, torch.float32), dev(plan_off, torch.int64),
                              rt.make_params(batch.params), out, ws))
    torch.cuda.synchronize()
    assert hz.device_status(ws) == 0
    return hz._np(out)


@pytest.mark.parametrize("d", [64, 1280])
@pytest.mark.parametrize("r", [17, 32, 33, 64])
def test_merge_uses_every_bit_of_the_plan(r, d):
    """Kept rows of zeros, pruned ones of +1 and -1 whose entries of a plan row differ in the last of their 24 bits: the
    merged row is that bit.  Every sum on the way to it is a whole number of them below 2^24, so it is exact."""
    B, n = 24, 400
    m = n - r
    image = np.zeros((n, d), np.float32)
    image[m:] = np.where(np.arange(r) % 2 == 0, 1.0, -1.0)[:, None]
    plan = np.zeros((m, r), np.float32)
    j = 2 * (np.arange(m) % (r // 2))                   # rows take the pairs of pruned tokens in turns
    plan[np.arange(m), j] = 0.5 + 2.0 ** -10 + 2.0 ** -23
    plan[np.arange(m), j + 1] = 0.5 + 2.0 ** -10
    for ratio in (0.84, 0.999):
        out = _merge_alone([image] * B, [n] * B, [m] * B, np.tile(plan.ravel(), B), alpha=1.0, ratio=ratio)
        assert (synth.bf16_bits_to_f32(out) == 2.0 ** -23).all(), (r, d, ratio)


def test_staged_merge_takes_its_kernel_from_the_counts():
    """The retention in the parameters says nothing about counts of the caller's own: whatever it is, the same kernel
    (the same bits: the kernels add up in different orders)."""
    rng = np.random.default_rng(61)
    for counts, r in (([400] * 20, 64), ([200, 400] * 4, 40), ([400] * 40 + [300] * 20, 33)):
        keep = [n - r for n in counts]
        tokens = [rng.standard_normal((n, 256)).astype(np.float32) for n in counts]
        plan = rng.random(sum(m * r for m in keep), dtype=np.float32)
        outs = [_merge_alone(tokens, counts, keep, plan, ratio=ratio) for ratio in (0.84, 0.3, 0.999)]
        np.testing.assert_array_equal(outs[0], outs[1])
        np.testing.assert_array_equal(outs[0], outs[2])


# ------------------------------------------------------------------ parameter sweeps
@pytest.mark.parametrize("override", [
    dict(eps=1.0, iters=100),           # the literal text of Appendix C
    dict(alpha=0.0),                    # pure pruning
    dict(z=1.0),                        # dustbin as attractive as a perfect match
    dict(z=0.0, alpha=0.5),
    dict(iters=0),
    dict(iters=1),
    dict(ratio=0.5),
    dict(ratio=0.25, iters=20),         # more pruned than kept
    dict(eps=0.0034, iters=30),         # the kernel matrix's exponents down to -588: the accepted range's end
])
def test_parameter_variants_c2_subset(override):
    batch = synth.gen_batch(2, images=range(4))
    params = dict(batch.params, **override)
    s = hz.run_staged(batch, params)
    rep = hz.compare_batch(batch, s, params, staged=True)
    _log(rep, f"c2 {override}")
    if override.get("alpha") == 0.0:
        for b in range(batch.batch):
            lo = int(batch.offsets[b])
            m = int(s["keep"][b])
            rows = batch.tokens[lo + s["sel"][lo:lo + m]]
            o0 = int(s["out_offsets"][b])
            np.testing.assert_array_equal(s["out"][o0:o0 + m], rows)


# ------------------------------------------------ variance selection metric (Table 7)
def _shifted_batch(dtype, seed, counts=(150, 64, 256, 1, 2), d=1152, **params):
    """Tokens with per-token feature shifts of varying size, so that the l2 norm and
    the variance rank them differently."""
    rng = np.random.default_rng(seed)
    imgs = []
    for c in counts:
        x = rng.standard_normal((c, d)) * rng.lognormal(0, 0.4, size=(c, 1))
        x += rng.standard_normal((c, 1)) * rng.choice([0.0, 0.5, 3.0], size=(c, 1))
        imgs.append(x.astype(np.float32))
    dens = rng.uniform(0.1, 0.9, len(counts)).astype(np.float32)
    p = dict(synth.DEFAULT_PARAMS, iters=20, metric=1)
    p.update(params)
    return synth.pack(0, dtype, imgs, dens, p)


@pytest.mark.parametrize("dtype,d", [("bf16", 1152), ("f32", 1152), ("bf16", 72), ("f32", 2048)])
def test_variance_metric_matches_the_oracle(dtype, d):
    batch = _shifted_batch(dtype, 77, d=d, ratio=0.7)
    s = hz.run_staged(batch, batch.params)
    rep = hz.compare_batch(batch, s, batch.params, staged=True)
    _log(rep, f"variance {dtype} D={d}")
    f = hz.run_prune(batch)
    for k in ("out_offsets", "keep", "sel", "pair"):
        np.testing.assert_array_equal(f[k], s[k])
    rows = int(s["out_offsets"][-1])
    np.testing.assert_array_equal(f["out"][:rows], s["out"][:rows])
    # the metric does change what is kept on this input
    l2 = hz.run_staged(batch, dict(batch.params, metric=0))
    assert not np.array_equal(l2["sel"], s["sel"])


def test_variance_metric_with_dynamic_ratio_on_clustered_pages():
    batch = synth.gen_batch(3, images=range(6))
    params = dict(batch.params, metric=1)
    f = hz.run_prune(batch, params)
    rep = hz.compare_batch(batch, f, params, staged=False)
    _log(rep, "c3 variance metric")


# ------------------------------------------------------------------------ edge cases
def _random_batch(counts, d, dtype, seed, dynamic=0, **params):
    rng = np.random.default_rng(seed)
    imgs = [(rng.standard_normal((c, d)) * rng.lognormal(0, 0.5, size=(c, 1))).astype(np.float32) for c in counts]
    dens = rng.uniform(0.1, 0.9, len(counts)).astype(np.float32)
    p = dict(synth.DEFAULT_PARAMS, iters=20, dynamic=dynamic)
    p.update(params)
    return synth.pack(0, dtype, imgs, dens, p)


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_degenerate_sizes(dtype):
    batch = _random_batch([0, 1, 2, 3, 0, 7, 1], 64, dtype, seed=1, dynamic=1, phi_hi=0.3)
    f = hz.run_prune(batch)
    assert f["rc"] == 0 and f["status"] == 0
    _log(hz.compare_batch(batch, f), f"degenerate {dtype}")
    s = hz.run_staged(batch)
    hz.compare_batch(batch, s, staged=True)
    assert f["keep"][0] == 0 and f["keep"][1] == 1 and f["keep"][4] == 0


def test_empty_batch_and_all_empty_images():
    b0 = synth.pack(0, "bf16", [], [], dict(synth.DEFAULT_PARAMS))
    f = hz.run_prune(b0)
    assert f["rc"] == 0 and list(f["out_offsets"]) == [0]
    b1 = _random_batch([0, 0, 0], 64, "bf16", seed=2)
    f = hz.run_prune(b1)
    assert f["rc"] == 0 and list(f["out_offsets"]) == [0, 0, 0, 0] and list(f["keep"]) == [0, 0, 0]


def test_nothing_pruned_passes_through():
    batch = _random_batch([33, 64], 128, "bf16", seed=3, ratio=1.0)
    f = hz.run_prune(batch)
    assert list(f["keep"]) == [33, 64]
    np.testing.assert_array_equal(f["out"][:97], batch.tokens)
    hz.compare_batch(batch, f)


@pytest.mark.parametrize("d,dtype", [(8, "bf16"), (4, "f32"), (72, "bf16"), (1288, "bf16"), (2048, "bf16"), (4096, "f32")])
def test_other_widths(d, dtype):
    batch = _random_batch([40, 17], d, dtype, seed=4, ratio=0.7)
    s = hz.run_staged(batch)
    _log(hz.compare_batch(batch, s, staged=True), f"width {d} {dtype}")


def test_identical_tokens_and_equal_norms():
    rng = np.random.default_rng(6)
    t = rng.standard_normal(64).astype(np.float32)
    same = np.tile(t, (20, 1))
    # all scores equal: the lowest indices are kept
    batch = synth.pack(0, "bf16", [same], [0.5], dict(synth.DEFAULT_PARAMS, iters=10, ratio=0.5))
    f = hz.run_prune(batch)
    assert list(f["sel"][:10]) == list(range(10))
    # every column of the plan is uniform: all kept rows tie, rank 0 wins
    assert (f["pair"][10:20] == 0).all()
    hz.compare_batch(batch, f)
    # equal norms, different directions
    u = rng.standard_normal((24, 64))
    u /= np.linalg.norm(u, axis=1, keepdims=True)
    batch = synth.pack(0, "f32", [u.astype(np.float32)], [0.5], dict(synth.DEFAULT_PARAMS, iters=10, ratio=0.5))
    hz.compare_batch(batch, hz.run_prune(batch))


@pytest.mark.parametrize("n,keep", [(600, 300), (600, 1), (600, 600), (600, 599), (1500, 777), (3000, 2048),
                                    (513, 256)])
def test_selection_on_long_images_with_many_equal_scores(n, keep):
    """Long images (the selection threshold is then found by radix passes over the
    keys) with scores that repeat: groups of identical tokens, a few distinct ones.
    Ties go to the lowest indices, exactly as the oracle's stable order does."""
    rng = np.random.default_rng(n + keep)
    protos = rng.standard_normal((7, 64)).astype(np.float32) * rng.lognormal(0, 0.5, size=(7, 1)).astype(np.float32)
    x = protos[rng.integers(0, 7, size=n)]
    x[rng.integers(0, n, size=5)] *= 3.0
    batch = synth.pack(0, "bf16", [x], [0.5], dict(synth.DEFAULT_PARAMS, iters=2, ratio=0.5))
    s = hz.run_staged(batch, keep_counts_in=[keep])
    assert int(s["keep"][0]) == keep
    X = orc.widen(batch.tokens, "bf16")
    ref = orc.prune_image(X, 0.5, orc.Params.from_dict(batch.params), keep_count=keep)
    np.testing.assert_array_equal(s["sel"][:keep], ref.kept)
    np.testing.assert_array_equal(s["sel"][keep:], ref.prop)


def test_zero_norm_tokens():
    rng = np.random.default_rng(7)
    x = rng.standard_normal((16, 64)).astype(np.float32)
    x[3] = 0
    x[9] = 0
    batch = synth.pack(0, "bf16", [x], [0.2], dict(synth.DEFAULT_PARAMS, iters=10, dynamic=1, phi_hi=0.1, ratio_min=0.5))
    f = hz.run_prune(batch)
    assert np.isfinite(synth.bf16_bits_to_f32(f["out"][: f["keep"][0]])).all()
    hz.compare_batch(batch, f)
    s = hz.run_staged(batch)
    hz.compare_batch(batch, s, staged=True)


def test_explicit_keep_counts():
    batch = _random_batch([30, 50, 12], 64, "bf16", seed=8)
    s = hz.run_staged(batch, keep_counts_in=[10, 50, 200])
    assert list(s["keep"]) == [10, 50, 12]          # clamped to N


def test_explicit_keep_counts_override_the_dynamic_bound():
    """Kept counts given by the caller can prune far more than the dynamic clamp
    would allow: the staged calls must not size anything from that clamp."""
    batch = synth.gen_batch(3, images=range(2))          # 400 tokens, dynamic parameters
    keep_in = [120, 150]                                 # 280 and 250 pruned tokens
    s = hz.run_staged(batch, keep_counts_in=keep_in)
    assert list(s["keep"][:2]) == keep_in
    p = orc.Params.from_dict(batch.params)
    for b in range(2):
        lo, hi = int(batch.offsets[b]), int(batch.offsets[b + 1])
        ref = orc.prune_image(orc.widen(batch.tokens[lo:hi], batch.dtype), float(batch.density[b]), p,
                              keep_count=keep_in[b])
        np.testing.assert_array_equal(s["sel"][lo:lo + keep_in[b]], ref.kept)
        po = int(s["plan_offsets"][b])
        S_g = s["scores"][po:po + ref.m * ref.r].reshape(ref.m, ref.r)
        assert np.abs(S_g - ref.S).max() <= hz.SCORE_ATOL
        o0 = int(s["out_offsets"][b])
        got = synth.bf16_bits_to_f32(s["out"][o0:o0 + ref.m]).astype(np.float64)
        assert np.abs(got - ref.merged).max() <= 0.5 * 2.0 ** -7 * np.abs(ref.merged).max() + 1e-6


def test_largest_supported_image():
    batch = _random_batch([8192], 64, "bf16", seed=9, ratio=0.97, iters=3)
    f = hz.run_prune(batch)
    assert f["rc"] == 0 and f["status"] == 0
    _log(hz.compare_batch(batch, f), "N=8192")


# ------------------------------------------------------------------ device-side errors
def test_bad_offsets_set_the_status_word_and_touch_nothing():
    batch = _random_batch([10, 12], 64, "bf16", seed=10)
    for bad, flag in (([0, 12, 10], rt.RTP_DEV_BAD_OFFSETS), ([1, 10, 22], rt.RTP_DEV_BAD_OFFSETS),
                      ([0, 10, 21], rt.RTP_DEV_BAD_OFFSETS)):
        b2 = synth.Batch(0, "bf16", batch.tokens, np.array(bad, dtype=np.int32), batch.density,
                         batch.params, [0, 1])
        db = rt.upload(b2)
        db.total_tokens, db.max_tokens = 22, 12
        ws = rt.alloc_workspace(db)
        out = torch.full((22, 64), 3.0, dtype=torch.bfloat16, device="cuda:0")
        off = torch.full((3,), -7, dtype=torch.int32, device="cuda:0")
        rc = rt.rtprune_prune(db, None, rt.make_params(batch.params), out, off, None, None, None, None, ws)
        torch.cuda.synchronize()
        assert rc == 0
        assert hz.device_status(ws) & flag
        assert (off.cpu().numpy() == -7).all() and (out.float().cpu().numpy() == 3.0).all()
    # an image longer than max_tokens
    db = rt.upload(batch)
    db.max_tokens = 11
    ws = rt.alloc_workspace(db)
    out = torch.zeros((22, 64), dtype=torch.bfloat16, device="cuda:0")
    off = torch.full((3,), -7, dtype=torch.int32, device="cuda:0")
    rc = rt.rtprune_prune(db, None, rt.make_params(batch.params), out, off, None, None, None, None, ws)
    torch.cuda.synchronize()
    assert rc == 0 and hz.device_status(ws) & rt.RTP_DEV_IMAGE_TOO_LONG
    assert (off.cpu().numpy() == -7).all()


def test_non_default_stream():
    batch = synth.gen_batch(2, images=range(3))
    ref = hz.run_prune(batch)
    st = torch.cuda.Stream()
    with torch.cuda.stream(st):
        got = hz.run_prune(batch)
    np.testing.assert_array_equal(ref["out"], got["out"])


def test_profile_records_per_kernel_and_can_be_restricted_to_one():
    """The measurement aids: one record per launch group while enabled, one kernel's alone on
    request, nothing once disabled; the results of the call do not change."""
    import torch
    batch = synth.gen_batch(2, images=range(4))
    plain = hz.run_prune(batch)
    rt.rtprune_profile_enable(1)
    try:
        f = hz.run_prune(batch)
        torch.cuda.synchronize()
        rc, rows = rt.rtprune_profile_summary()
        assert rc == rt.RTP_OK
        names = {r["kernel"] for r in rows}
        assert {"k_norms", "k_select", "k_scores", "k_sinkhorn_regs", "k_merge"} <= names
        # the fused call checks the layout in the norm pass and leaves the batch-wide sums to
        # the score pass: neither has a launch of its own
        assert "k_prepare" not in names and "k_scan" not in names
        assert all(r["launches"] >= 1 and r["total_ms"] > 0 for r in rows)
        rt.rtprune_profile_enable(1)                    # discards the records
        assert rt.rtprune_profile_only("k_merge") == rt.RTP_OK
        g = hz.run_prune(batch)
        torch.cuda.synchronize()
        rc, rows = rt.rtprune_profile_summary()
        assert rc == rt.RTP_OK and [r["kernel"] for r in rows] == ["k_merge"] and rows[0]["launches"] == 1
    finally:
        rt.rtprune_profile_only(None)
        rt.rtprune_profile_enable(0)
    hz.run_prune(batch)
    rc, rows = rt.rtprune_profile_summary()
    assert rc == rt.RTP_OK and rows == []
    for other in (f, g):
        np.testing.assert_array_equal(other["out"], plain["out"])
        np.testing.assert_array_equal(other["pair"], plain["pair"])
