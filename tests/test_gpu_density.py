"""GPU parity of the textual-density kernel (Eq. 8, Appendix B) against the
oracle: edge counts are integers, so rho and rho_k must be bit-exact."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

from oracle import rtprune_oracle as orc  # noqa: E402
from paper_2605_00392_amd import rtprune as rt  # noqa: E402
from paper_2605_00392_amd import synth  # noqa: E402


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    rt.load_library()


def run_density(pages, patch_h, patch_w, tau, max_h=None, max_w=None, want_patches=True, pad=0):
    """pages: list of uint8 arrays [H, W, 3]; returns (rc, status, rho[B], rho_k list)."""
    dev = "cuda:0"
    B = len(pages)
    hs = np.array([p.shape[0] for p in pages], dtype=np.int32)
    ws_ = np.array([p.shape[1] for p in pages], dtype=np.int32)
    sizes = np.array([p.size + pad for p in pages], dtype=np.int64)
    poff = np.zeros(B + 1, dtype=np.int64)
    poff[1:] = np.cumsum(sizes)
    flat = np.zeros(max(int(poff[-1]), 1), dtype=np.uint8)
    for b, p in enumerate(pages):
        flat[poff[b]:poff[b] + p.size] = p.ravel()
    npatch = (hs // patch_h) * (ws_ // patch_w)
    pto = np.zeros(B + 1, dtype=np.int32)
    pto[1:] = np.cumsum(npatch)
    mh = int(hs.max()) if max_h is None and B else (max_h or 0)
    mw = int(ws_.max()) if max_w is None and B else (max_w or 0)
    rc, nbytes = rt.rtprune_text_density_workspace_bytes(B, mh, mw, patch_h, patch_w)
    assert rc == 0, rc
    wsb = torch.empty(nbytes, dtype=torch.uint8, device=dev)
    t = lambda a: torch.from_numpy(a).to(dev)
    d_pix, d_off, d_h, d_w, d_pto = t(flat), t(poff), t(hs if B else np.zeros(1, np.int32)), t(ws_ if B else np.zeros(1, np.int32)), t(pto)
    rho = torch.full((max(B, 1),), -7.0, dtype=torch.float32, device=dev)
    rho_k = torch.full((max(int(pto[-1]), 1),), -7.0, dtype=torch.float32, device=dev)
    rc = rt.rtprune_text_density(d_pix, d_off, d_h, d_w, B, mh, mw, patch_h, patch_w, tau, rho,
                                 rho_k if want_patches else None, d_pto if want_patches else None, wsb)
    torch.cuda.synchronize()
    status = int(wsb[:4].view(torch.int32).item()) if (rc == 0 and B) else 0
    rk = rho_k.cpu().numpy()
    return rc, status, rho.cpu().numpy()[:B], [rk[pto[b]:pto[b + 1]] for b in range(B)]


def check(pages, patch_h, patch_w, tau, **kw):
    rc, status, rho, rho_k = run_density(pages, patch_h, patch_w, tau, **kw)
    assert rc == 0 and status == 0
    for b, p in enumerate(pages):
        want, want_k = orc.text_density(p, patch_h, patch_w, tau)
        assert rho[b] == want, (b, rho[b], want)
        np.testing.assert_array_equal(rho_k[b], want_k)
    return rho


def test_large_mode_pages_bit_exact():
    pages = [synth.gen_page(i, 1280) for i in range(6)]
    rho = check(pages, 64, 64, 0.2)
    assert rho.min() > 0.0 and rho.max() < 0.6
    print("\n[density large] rho =", np.round(rho, 4).tolist(), flush=True)


def test_all_native_modes_and_thresholds():
    for mode, side in synth.PAGE_MODES.items():
        pages = [synth.gen_page(100 + i, side) for i in range(2)]
        for tau in (0.1, 0.2, 0.3, 0.5):          # the values of the paper's threshold ablation
            check(pages, synth.PATCH_PIXELS, synth.PATCH_PIXELS, tau)


def test_ragged_batch_of_tiles_and_global_views():
    # a tiled page: 640 x 640 local tiles and a 1024 x 1024 global view, different sizes in one batch
    pages = [synth.gen_page(200, 640), synth.gen_page(201, 1024), synth.gen_page(202, 512), synth.gen_page(203, 640)]
    check(pages, 64, 64, 0.2)
    check(pages, 64, 64, 0.2, pad=5)             # page starts that are not 4-byte aligned


def test_random_noise_odd_shapes_and_patch_sizes():
    rng = np.random.default_rng(40)
    for (h, w, ph, pw) in ((34, 51, 17, 17), (48, 36, 6, 9), (14, 14, 14, 14), (7, 5, 7, 5), (1, 1, 1, 1),
                           (96, 4100, 32, 4100), (64, 64, 64, 64)):
        img = rng.integers(0, 256, size=(h, w, 3)).astype(np.uint8)
        for tau in (0.05, 0.2, 1.0, 2.5):
            check([img], ph, pw, tau)


def test_exact_threshold_cases():
    g = np.zeros((8, 8, 3), dtype=np.uint8)
    g[:, 4:] = 255                                # G = 4.0 exactly on two columns
    rho = check([g], 8, 8, 4.0)
    assert rho[0] == np.float32(16 / 64)
    rho = check([g], 8, 8, float(np.nextafter(np.float32(4.0), np.float32(5))))
    assert rho[0] == 0.0
    rho = check([g], 8, 8, 0.0)                   # tau = 0: every pixel is an edge
    assert rho[0] == 1.0
    flat = np.full((64, 64, 3), 200, dtype=np.uint8)
    assert check([flat], 16, 16, 0.2)[0] == 0.0
    # gradients sitting near the threshold: small steps of every size
    rng = np.random.default_rng(41)
    base = rng.integers(100, 104, size=(64, 64, 1)).astype(np.uint8)
    img = np.repeat(base, 3, axis=2) + rng.integers(0, 14, size=(64, 64, 3)).astype(np.uint8)
    for tau in (0.04, 0.08, 0.12, 0.16, 0.2):
        check([img], 8, 8, tau)


@pytest.mark.parametrize("pad", [0, 1, 2, 3])
def test_patches_of_whole_segments_at_the_edges_of_bands(pad):
    """Patch widths that are a multiple of 64: pages of one patch, of bands of 256 columns and one patch either
    side, noise (saturated bytes among it) whose gradients lie on both sides of every threshold."""
    rng = np.random.default_rng(42 + pad)
    for pw, ph, sizes in ((64, 64, ((64, 64), (128, 192), (64, 256), (64, 320), (128, 576))),
                          (64, 1, ((1, 64), (2, 256), (3, 320))), (128, 5, ((5, 128), (10, 384))), (320, 7, ((14, 320), (7, 640)))):
        pages = [rng.integers(0, 256, size=(h, w, 3)).astype(np.uint8) for h, w in sizes]
        pages += [(255 * rng.integers(0, 2, size=(h, w, 3))).astype(np.uint8) for h, w in sizes]
        pages += [(100 + rng.integers(0, 20, size=(h, w, 3))).astype(np.uint8) for h, w in sizes]
        for tau in (0.0, 0.05, 0.2, 1.0, 4.0):
            check(pages, ph, pw, tau, pad=pad)


@pytest.mark.parametrize("pad", [0, 1, 2, 5])
def test_patches_of_whole_words_at_the_edges_of_bands(pad):
    """Patch widths that are a multiple of 4 but not of 64: the register-window kernel, with bands of 248 columns, on pages
    that start at a word and that do not (its byte path)."""
    rng = np.random.default_rng(46 + pad)
    for pw, ph, sizes in ((20, 10, ((10, 20), (20, 240), (30, 260), (20, 520))), (248, 4, ((4, 248), (8, 496), (4, 744))),
                          (4, 1, ((1, 4), (3, 252), (2, 300)))):
        pages = [rng.integers(0, 256, size=(h, w, 3)).astype(np.uint8) for h, w in sizes]
        pages += [(100 + rng.integers(0, 20, size=(h, w, 3))).astype(np.uint8) for h, w in sizes]
        for tau in (0.0, 0.05, 0.2, 1.0):
            check(pages, ph, pw, tau, pad=pad)


@pytest.mark.parametrize("ph,copies", [(64, 20), (64, 30), (64, 50), (64, 75), (40, 20), (23, 50)])
def test_patch_rows_shared_by_several_waves(ph, copies):
    """Batches in which seven, five, three and two waves share a patch row of 64 (most of these do not divide it: the last
    has fewer), and one of 40 and of 23 rows: the count of every page is that of its first copy and of the oracle."""
    rng = np.random.default_rng(47)
    h = 5 * ph
    pages = [rng.integers(0, 256, size=(h, 320, 3)).astype(np.uint8), synth.gen_page(500, 640)[:h, :320].copy(),
             (100 + rng.integers(0, 20, size=(h, 320, 3))).astype(np.uint8), synth.gen_page(501, 640)[100:100 + h, 64:384].copy()]
    rc, status, rho, rho_k = run_density(pages * copies, ph, 64, 0.2)
    assert rc == 0 and status == 0
    for b in range(4 * copies):
        if b < 4:
            want, want_k = orc.text_density(pages[b], ph, 64, 0.2)
            assert rho[b] == want, (b, rho[b], want)
            np.testing.assert_array_equal(rho_k[b], want_k)
        else:
            np.testing.assert_array_equal(rho_k[b], rho_k[b % 4])
            assert rho[b] == rho[b % 4]


def test_empty_batch_and_optional_outputs():
    rc, status, rho, _ = run_density([], 64, 64, 0.2)
    assert rc == 0
    pages = [synth.gen_page(300, 512)]
    rc, status, rho, _ = run_density(pages, 64, 64, 0.2, want_patches=False)
    assert rc == 0 and status == 0 and rho[0] == orc.text_density(pages[0], 64, 64, 0.2)[0]


def test_bad_geometry_sets_the_status_word():
    img = np.zeros((60, 64, 3), dtype=np.uint8)   # height not a multiple of the patch
    rc, status, rho, _ = run_density([img], 64, 64, 0.2, max_h=64, max_w=64)
    assert rc == 0 and status & rt.RTP_DEV_BAD_IMAGE and rho[0] == -7.0
    img = np.zeros((128, 64, 3), dtype=np.uint8)  # taller than the stated maximum
    rc, status, rho, _ = run_density([img], 64, 64, 0.2, max_h=64, max_w=64)
    assert rc == 0 and status & rt.RTP_DEV_BAD_IMAGE and rho[0] == -7.0


def test_density_feeds_the_dynamic_ratio():
    # pages -> rho on the device -> rtprune_dynamic_ratio, against the oracle end to end
    batch = synth.gen_batch(3, images=range(4))
    pages = [synth.gen_page(400 + i, 1280) for i in range(4)]
    rc, status, rho, _ = run_density(pages, 64, 64, 0.2)
    assert rc == 0 and status == 0
    db = rt.upload(batch)
    ws = rt.alloc_workspace(db)
    dev = "cuda:0"
    phi = torch.zeros(4, dtype=torch.float32, device=dev)
    ratio = torch.zeros(4, dtype=torch.float32, device=dev)
    keep = torch.zeros(4, dtype=torch.int32, device=dev)
    p = rt.make_params(batch.params)
    rt.check(rt.rtprune_dynamic_ratio(db, torch.from_numpy(rho).to(dev), p, phi, ratio, keep, ws))
    torch.cuda.synchronize()
    op = orc.Params.from_dict(batch.params)
    for b in range(4):
        X = orc.widen(batch.tokens[batch.offsets[b]:batch.offsets[b + 1]], "bf16")
        want_rho, _ = orc.text_density(pages[b], 64, 64, 0.2)
        ret = orc.dynamic_retention(orc.inter_token_similarity(X), want_rho, op)
        assert abs(float(ratio[b].item()) - float(ret)) <= 1e-6
        assert int(keep[b].item()) == orc.kept_count(ret, 400)
