"""GPU parity of edge_importance against the CPU oracle (through the C ABI).

Sizes the oracle finishes in seconds that still span several strips (248
output columns each), several bands and ragged tails, plus full-size batched
workloads checked on sampled views in the launch configuration the benchmark
times.
"""
import numpy as np
import pytest

import oracle
import synth
from parity import check_batch, compare_view, gpu_edge, view_map

pytestmark = pytest.mark.gpu

PRECS = ["fp32", "fp16", "bf16"]
BATCHED_FORMS = ["staged", "persistent"]


def small_batch(in_align=1, out_align=1):
    """Ragged views around every strip/band/alignment boundary."""
    sizes = [(3, 3), (4, 5), (7, 3), (3, 9), (247, 9), (248, 17), (249, 31), (252, 8), (253, 12),
             (256, 64), (257, 300), (500, 70), (744, 33), (1001, 13), (61, 513)]
    imgs = [synth.image(40 + k, w, h, n_poly=6, texture=(k % 2 == 0)) for k, (w, h) in enumerate(sizes)]
    return synth.pack_views(imgs, in_align=in_align, out_align=out_align)


@pytest.mark.parametrize("precision", PRECS)
def test_single_256x192_view(precision):
    w = synth.workload("view_256x192")
    vb = w.render(in_align=256, out_align=64)
    for form in ("plain", "staged", "persistent"):
        st = check_batch(vb, precision, form)
        print(precision, form, st)


@pytest.mark.parametrize("form", BATCHED_FORMS + ["unfused"])
@pytest.mark.parametrize("precision", PRECS)
def test_ragged_views_unaligned(precision, form):
    vb = small_batch()
    st = check_batch(vb, precision, form)
    print(precision, form, sum(s["mismatch"] for s in st), max(s["scaled_err"] for s in st))


@pytest.mark.parametrize("form", BATCHED_FORMS)
@pytest.mark.parametrize("seg_rows,wg_waves", [(8, 1), (16, 2), (32, 4), (64, 8), (128, 4), (24, 2)])
def test_tile_shapes(seg_rows, wg_waves, form):
    vb = small_batch(in_align=16, out_align=4)
    check_batch(vb, "fp32", form, seg_rows=seg_rows, wg_waves=wg_waves)


@pytest.mark.parametrize("precision", PRECS)
def test_random_view_sizes(precision):
    """48 views of seeded random sizes, from 3x3 up to several strips wide
    and bands tall, at random alignments: many short last bands in the
    launch's per-XCD order, every border case of the strips."""
    rng = np.random.default_rng(2024)
    sizes = [(int(rng.integers(3, 700)), int(rng.integers(3, 260))) for _ in range(48)]
    imgs = [synth.image(500 + k, w, h, n_poly=5, texture=bool(k % 2)) for k, (w, h) in enumerate(sizes)]
    vb = synth.pack_views(imgs, in_align=int(rng.integers(1, 17)), out_align=int(rng.integers(1, 5)))
    for form, kw in (("staged", {}), ("staged", {"seg_rows": 16, "wg_waves": 2}), ("plain", {})):
        st = check_batch(vb, precision, form, **kw)
        print(precision, form, kw, sum(s["mismatch"] for s in st), max(s["scaled_err"] for s in st))


def test_adversarial_images():
    H, W = 40, 300
    imgs = []
    im = np.zeros((H, W, 3), np.uint8)
    imgs.append(im.copy())                                   # constant: nothing survives
    im[:, 150:] = 255
    imgs.append(im.copy())                                   # ideal step
    imgs.append(np.ascontiguousarray(np.transpose(imgs[-1][:, :H], (1, 0, 2))))
    ramp = np.zeros((H, W, 3), np.uint8)
    ramp[:] = (np.arange(W) % 256).astype(np.uint8)[None, :, None]
    imgs.append(ramp)
    yy, xx = np.mgrid[0:H, 0:W]
    imgs.append(np.repeat((((yy // 2 + xx // 3) % 2) * 200 + 20).astype(np.uint8)[..., None], 3, 2))
    imgs.append(np.random.default_rng(0).integers(0, 256, (H, W, 3), dtype=np.uint8))
    imgs.append(np.random.default_rng(1).integers(100, 103, (H, W, 3), dtype=np.uint8))
    vb = synth.pack_views(imgs, in_align=1, out_align=1)
    for p in PRECS:
        for form in BATCHED_FORMS:
            check_batch(vb, p, form)


def test_step_edge_ridge_exact():
    im = np.zeros((37, 520, 3), np.uint8)
    im[:, 261:] = 255
    vb = synth.pack_views([im])
    E, _, nsv = gpu_edge(vb, "fp32")
    Em = view_map(E, vb, 0)
    assert (Em[:, 260] == 1.0).all() and (np.delete(Em, 260, axis=1) == 0).all() and nsv[0] == 37


@pytest.mark.parametrize("precision", PRECS)
def test_forms_equal_and_deterministic(precision):
    """Every launch form gives the same bits; repeated calls reuse the plan
    (whose counters, histograms and queue each call restores)."""
    vb = small_batch(in_align=16, out_align=4)
    a = gpu_edge(vb, precision, "staged")
    others = [gpu_edge(vb, precision, "plain"), gpu_edge(vb, precision, "persistent"),
              gpu_edge(vb, precision, "persistent", reps=4), gpu_edge(vb, precision, "staged", reps=3),
              gpu_edge(vb, precision, "unfused"), gpu_edge(vb, precision, "unfused", reps=2)]
    for y in others:
        for u, v in zip(a, y):
            assert (u == v).all()


def test_permuting_views_permutes_outputs():
    vb = small_batch(in_align=16, out_align=4)
    perm = list(range(vb.n))[::-1]
    vp = synth.pack_views([vb.view(v) for v in perm], in_align=7, out_align=3)
    a, _, _ = gpu_edge(vb, "fp16")
    b, _, _ = gpu_edge(vp, "fp16")
    for k, v in enumerate(perm):
        assert (view_map(a, vb, v) == view_map(b, vp, k)).all()


def test_single_1297x840_view_full_oracle():
    w = synth.workload("view_1297x840")
    vb = w.render(in_align=256, out_align=64)
    for p, form in zip(PRECS, ("plain", "staged", "persistent")):
        st = check_batch(vb, p, form)
        print(w.name, p, form, st)


@pytest.mark.parametrize("name,precisions,sample", [("views200_w1000_1560", ["fp16", "fp32"], [0, 57, 199]),
                                                    ("views150_2473x1643_mixed", ["fp16", "bf16"], [0, 1, 148, 149]),
                                                    ("step_views300_las3m", ["bf16"], [0, 150, 299])])
def test_full_size_workloads_sampled(name, precisions, sample):
    """Every view of the full workload goes through one persistent launch (the
    form the benchmark times); sampled views are checked against the oracle
    pixel by pixel, and the staged form must give the same bits."""
    w = synth.workload(name)
    vb = w.render()
    refs = {v: oracle.edge_view(vb.view(v)) for v in sample}
    for p in precisions:
        E, med, nsv = gpu_edge(vb, p, "persistent")
        for v in sample:
            st = compare_view(view_map(E, vb, v), refs[v], p, med[v], nsv[v])
            print(f"{name} {p} view {v}", st)
        assert (nsv > 0).all() and (med > 0).all()
        E2, med2, nsv2 = gpu_edge(vb, p, "staged")
        assert (E2 == E).all() and (med2 == med).all() and (nsv2 == nsv).all()


@pytest.mark.parametrize("precision", PRECS)
def test_status_word_and_forced_persistent_timeout(precision, monkeypatch):
    """Every form sets the caller's status word to IGSP_OK. The persistent
    form reports IGSP_ERR_TIMEOUT when its bounded waits give up: the host
    forces that here (IGSP_PERSIST_FORCE_TIMEOUT makes every wait give up
    after a few polls, so every kernel still exits), and the next call, with
    the normal bound, starts clean and matches the oracle again."""
    import torch

    import paper_2603_08661_amd as igsp

    vb = small_batch(in_align=16, out_align=4)
    dev = torch.device("cuda:0")
    img = torch.from_numpy(np.concatenate([vb.rgb, np.zeros(32, np.uint8)])).to(dev)
    out = torch.zeros(vb.out_floats, dtype=torch.float32, device=dev)
    status = torch.full((1,), 99, dtype=torch.int32, device=dev)
    views = (vb.widths, vb.heights, vb.in_offset, vb.out_offset)
    refs = [oracle.edge_view(vb.view(v)) for v in range(vb.n)]

    def run(form):
        status.fill_(99)
        igsp.edge_importance(img, views, out, precision=precision, batched=form, status=status)
        torch.cuda.synchronize()
        return int(status.item())

    def check():
        E = out.cpu().numpy()
        for v in range(vb.n):
            compare_view(view_map(E, vb, v), refs[v], precision)

    for form in ("plain", "staged", "persistent", "unfused"):
        assert run(form) == 0, form
        check()
    monkeypatch.setenv("IGSP_PERSIST_FORCE_TIMEOUT", "1")
    print("forcing the persistent form's waits to give up", flush=True)
    assert run("persistent") == -9
    monkeypatch.delenv("IGSP_PERSIST_FORCE_TIMEOUT")
    for _ in range(2):
        assert run("persistent") == 0
        check()


def test_more_geometries_than_the_plan_cache_holds():
    """Ten geometries, each called twice in interleaved order: the library
    keeps eight edge plans and frees the least recently used one when it
    builds another, so the second round rebuilds plans it evicted. Every map
    matches the oracle."""
    sizes = [(40 + 23 * k, 30 + 11 * k) for k in range(10)]
    batches = [synth.pack_views([synth.image(900 + k, w, h, n_poly=5, texture=True)], in_align=16, out_align=4)
               for k, (w, h) in enumerate(sizes)]
    refs = [oracle.edge_view(vb.view(0)) for vb in batches]
    for rnd in range(2):
        for k in (list(range(10)) if rnd == 0 else list(range(9, -1, -2)) + list(range(0, 10, 2))):
            E, med, nsv = gpu_edge(batches[k], "bf16", "staged")
            compare_view(view_map(E, batches[k], 0), refs[k], "bf16", med[0], nsv[0])


# (Views of this size take the short median chain in the plain and staged forms,
# which lists nothing: here only the unfused form reads the lists. Staged launches
# do from larger views on: test_fp32_candidate_list_cut_off.)
@pytest.mark.parametrize("form", ["plain", "staged", "unfused"])
def test_fp32_median_candidates_overflow_and_fit(form):
    """In launches over several views (staged, unfused), the second FP32
    refinement pass reads the first pass's candidate list (the survivors of
    the first histogram's median bucket) when it fits in the view's room
    (1/16 of its pixels, at least 256), else the map; the plain form's
    one-view launches always read the map. A striped view puts nearly every
    survivor in one bucket (the list overflows); a textured view of the same
    size does not. Every view matches the oracle."""
    H, W = 64, 600
    stripes = np.zeros((H, W, 3), np.uint8)
    stripes[:] = ((((np.arange(W) // 3) % 2) * 180) + 30).astype(np.uint8)[None, :, None]
    textured = synth.image(77, W, H, n_poly=8, texture=True)
    room = max(H * W // 16, 256)
    counts = []
    for im in (stripes, textured):
        o = oracle.edge_view(im)
        keep = o["keep"].astype(bool)
        bits = o["M"][keep].astype(np.float32).view(np.uint32)
        med = np.float32(o["Mmed"]).view(np.uint32)
        counts.append(int(((bits >> 16) == (med >> 16)).sum()))
    assert counts[0] > room >= counts[1], (counts, room)
    vb = synth.pack_views([stripes, textured, stripes], in_align=3, out_align=2)
    check_batch(vb, "fp32", form)


# (The short chain counts every value exactly and has no list: these are stripes
# with one and with very many values in the median's bucket for it.)
@pytest.mark.parametrize("form", ["plain", "staged"])
def test_fp32_candidate_list_without_room(form):
    """The short chain lists the median bucket's values with their counts
    (room: 1/16 of the view's pixels, at least 256). Stripes with one grey
    level of noise give more distinct values in that bucket than there is
    room for, so the selection reads the map; the view beside them has plain
    stripes (many survivors, few values) and lists them."""
    H, W = 64, 600
    flat = np.zeros((H, W, 3), np.uint8)
    flat[:] = ((((np.arange(W) // 3) % 2) * 180) + 30).astype(np.uint8)[None, :, None]
    noisy = flat + np.random.default_rng(5).integers(0, 2, flat.shape).astype(np.uint8)
    distinct = []
    for im in (flat, noisy):
        o = oracle.edge_view(im)
        bits = o["M"][o["keep"].astype(bool)].astype(np.float32).view(np.uint32)
        med = np.float32(o["Mmed"]).view(np.uint32)
        distinct.append(np.unique(bits[(bits >> 16) == (med >> 16)]).size)
    assert distinct[0] < 64 and distinct[1] > H * W // 16, distinct
    check_batch(synth.pack_views([noisy, flat, noisy], in_align=1, out_align=2), "fp32", form, reps=2)


# (688 chunks: FP32's guarded chain on both sides, FP16's long one; the chains'
# lines are taken by test_median_chains_on_either_side_of_their_lines.)
@pytest.mark.parametrize("precision", ["fp32", "fp16"])
@pytest.mark.parametrize("rows", [1376, 1377])
def test_short_and_long_median_chain(precision, rows):
    """688 element-wise chunks (8 strips x 1376 rows, 16 slots each) are the
    most the short chain takes of one view; one row more takes the long one.
    Both equal the unfused form, which always takes the long one, bit for bit."""
    vb = synth.pack_views([synth.image(61, 1984, rows, n_poly=20, texture=True)], in_align=16, out_align=4)
    a, ma, na = gpu_edge(vb, precision, "staged", reps=2)
    b, mb, nb = gpu_edge(vb, precision, "unfused")
    assert np.array_equal(a, b) and np.array_equal(ma, mb) and np.array_equal(na, nb) and na[0] > 0


@pytest.mark.parametrize("rows", [2500, 2499])
def test_fp32_wide_refinement_chunks(rows):
    """Two views of 8 strips x 2500 rows are 40000 slots, the fewest whose FP32
    refinement takes 128 slots per work-group; one row less takes 64. One view
    is textured (its second pass reads the candidate list), one striped (the
    list overflows, the pass reads the map). Both equal the persistent form
    bit for bit."""
    stripes = np.zeros((rows, 1984, 3), np.uint8)
    stripes[:] = ((((np.arange(1984) // 3) % 2) * 180) + 30).astype(np.uint8)[None, :, None]
    vb = synth.pack_views([synth.image(62, 1984, rows, n_poly=20, texture=True), stripes], in_align=16, out_align=4)
    a, ma, na = gpu_edge(vb, "fp32", "staged", reps=2)
    b, mb, nb = gpu_edge(vb, "fp32", "persistent")
    assert np.array_equal(a, b) and np.array_equal(ma, mb) and np.array_equal(na, nb) and (na > 0).all()


@pytest.mark.parametrize("precision", ["fp32", "fp16", "bf16"])
@pytest.mark.parametrize("seg_rows", [0, 8, 13, 64])
def test_ties_and_segment_remainders(precision, seg_rows):
    """Flat blocks, steps and stripes make magnitudes that equal a neighbour's
    (the tie rule decides, on a path of its own); heights from one to two
    rounds of the stencil's six rows past the segment give every remainder.
    All equal the unfused form, which always applies the whole rule."""
    rng = np.random.default_rng(31)
    imgs = []
    for h in range(64, 78):
        blocks = np.kron(rng.integers(0, 4, (h // 8 + 1, 40, 3)) * 60, np.ones((8, 7, 1), int))[:h, :270]
        imgs.append(blocks.astype(np.uint8))
    imgs += [np.ascontiguousarray(im.transpose(1, 0, 2)) for im in imgs[:3]]
    vb = synth.pack_views(imgs, in_align=1, out_align=3)
    a, ma, na = gpu_edge(vb, precision, "staged", seg_rows=seg_rows, reps=2)
    b, mb, nb = gpu_edge(vb, precision, "unfused")
    for v in range(vb.n):
        assert np.array_equal(view_map(a, vb, v), view_map(b, vb, v)), v
    assert np.array_equal(ma, mb) and np.array_equal(na, nb) and (na > 0).all()
    check_batch(vb, precision, "plain", views=[0, 13, 16])


@pytest.mark.parametrize("n_views", [1, 64, 65])
def test_fp32_short_chain_equal_and_distinct_values(n_views):
    """The short chain counts the median bucket's values after merging equal
    ones: 6-pixel stripes have one magnitude (thousands of candidates a chunk,
    all equal), with sensor noise they have thousands of different ones, and a
    textured view has a few. 64 views are the most that one FP32 launch counts
    this way. All equal the unfused form, which never does, bit for bit."""
    rng = np.random.default_rng(7)
    imgs = []
    for k in range(n_views):
        h, w = (300, 500) if k < 3 else (20 + k % 7, 30 + k % 5)
        im = np.zeros((h, w, 3)) + ((((np.arange(w) // 3) % 2) * 180) + 30)[None, :, None]
        if k % 3 != 1:
            im = im + rng.normal(0, 1.0, (h, w, 1))
        imgs.append(np.clip(np.rint(im), 0, 255).astype(np.uint8) if k % 3 != 2 else synth.image(70 + k, w, h, n_poly=10, texture=True))
    vb = synth.pack_views(imgs, in_align=1, out_align=4)
    a, ma, na = gpu_edge(vb, "fp32", "staged", reps=3)
    p, mp, np_ = gpu_edge(vb, "fp32", "plain", reps=2)
    b, mb, nb = gpu_edge(vb, "fp32", "unfused")
    assert np.array_equal(a, b) and np.array_equal(ma, mb) and np.array_equal(na, nb) and (na > 0).any()
    assert np.array_equal(p, b) and np.array_equal(mp, mb) and np.array_equal(np_, nb)


def test_heights_marched_alike_share_a_plan():
    """Segment heights of 8 to 12 rows are all marched as two rounds of six (this
    view fills more than 1.5 wavefronts per SIMD at six rows, so 10 is too): one
    plan, with one intermediate map, serves them. 13 rows take another."""
    import torch

    import paper_2603_08661_amd as igsp

    W, H = 2000, 1500
    dev = torch.device("cuda:0")
    img = torch.from_numpy(np.concatenate([synth.image(63, W, H, 30, True).reshape(-1), np.zeros(16, np.uint8)])).to(dev)
    views = ([W], [H], [0], [0])
    maps = {seg: torch.zeros(W * H, device=dev) for seg in (12, 8, 9, 10, 11, 13)}
    torch.cuda.synchronize()
    igsp.release_plans()
    free = {}
    for seg, out in maps.items():      # (no torch operation in between: they allocate too)
        igsp.edge_importance(img, views, out, precision="fp32", batched="staged", seg_rows=seg)
        torch.cuda.synchronize()
        free[seg] = torch.cuda.mem_get_info(dev)[0]
    assert free[8] == free[9] == free[10] == free[11] == free[12], free
    assert free[12] - free[13] >= 4 * W * H, free
    assert all(torch.equal(m, maps[12]) for m in maps.values())
    igsp.release_plans()


def _striped(w, h, rng=None):
    """6-pixel stripes of one contrast, with a grey level of sensor noise."""
    im = np.zeros((h, w, 3)) + ((((np.arange(w) // 3) % 2) * 180) + 30)[None, :, None]
    if rng is not None:
        im = im + rng.normal(0, 1.0, (h, w, 1))
    return np.clip(np.rint(im), 0, 255).astype(np.uint8)


def _in_median_bucket(im):
    """Survivors whose FP32 value shares the median's upper 16 bits."""
    o = oracle.edge_view(im)
    bits = o["M"][o["keep"].astype(bool)].astype(np.float32).view(np.uint32)
    return int((bits >> 16 == np.float32(o["Mmed"]).view(np.uint32) >> 16).sum())


@pytest.mark.parametrize("size,kinds", [((1736, 1150), "n"), ((1736, 1150), "t"), ((1736, 1150), "c"),
                                        ((1297, 840), "ntsc"), ((640, 480), "ntscntscntscntsc")])
def test_fp32_guarded_chain(size, kinds):
    """Views that take the guarded median chain together (more chunks than the
    short chain's line, fewer than the long one's): striped with noise and plain
    stripes (more than 128 survivors a chunk in the median's bucket: the refinement
    launch counts their last digit), textured (fewer: counted one by one) and
    constant (none). Every form gives the same bits, call after call."""
    w, h = size
    rng = np.random.default_rng(17)
    make = {"n": lambda k: _striped(w, h, rng), "s": lambda k: _striped(w, h),
            "t": lambda k: synth.image(170 + k, w, h, n_poly=20, texture=True), "c": lambda k: np.full((h, w, 3), 90, np.uint8)}
    imgs = [make[c](k) for k, c in enumerate(kinds)]
    chunks = -(-(-(-w // 248) * h) // 16)
    for im, c in list(zip(imgs, kinds))[:3]:
        if c != "c":
            assert (_in_median_bucket(im) > 128 * chunks) == (c != "t"), c
    vb = synth.pack_views(imgs, in_align=1, out_align=3)
    b, mb, nb = gpu_edge(vb, "fp32", "unfused")
    assert [n > 0 for n in nb] == [c != "c" for c in kinds]
    for form, reps in (("staged", 3), ("plain", 2), ("persistent", 1), ("staged", 1)):
        a, ma, na = gpu_edge(vb, "fp32", form, reps=reps)
        assert np.array_equal(a, b) and np.array_equal(ma, mb) and np.array_equal(na, nb), form


@pytest.mark.parametrize("precision,chunks", [("fp32", 360), ("fp32", 361), ("fp32", 700), ("fp32", 701),
                                              ("fp16", 510), ("fp16", 511)])
@pytest.mark.parametrize("noise", [False, True])
def test_median_chains_on_either_side_of_their_lines(precision, chunks, noise):
    """One view of 5 strips with the most chunks that a chain takes and one more,
    textured and striped with noise, against the unfused form (the long chain)."""
    w, h = 1240, 16 * chunks // 5
    assert -(-5 * h // 16) == chunks
    im = _striped(w, h, np.random.default_rng(19)) if noise else synth.image(180, w, h, n_poly=20, texture=True)
    vb = synth.pack_views([im], in_align=16, out_align=4)
    a, ma, na = gpu_edge(vb, precision, "staged", reps=2)
    b, mb, nb = gpu_edge(vb, precision, "unfused")
    assert np.array_equal(a, b) and np.array_equal(ma, mb) and np.array_equal(na, nb) and na[0] > 0


@pytest.mark.parametrize("sizes", [[(6000, 4000)], [(500, 400)] * 64])
def test_fp32_plans_hold_what_their_launches_use(sizes):
    """Beside a map of twice the size, an FP32 plan takes more memory than a BF16
    one only for what some launch of it uses: one large view neither lists its
    median's candidates nor counts values; 64 views that take the long chain
    together list candidates (1/16 of the pixels) and count values for one view at
    a time, in the plain form, not for all 64 (16 MiB)."""
    import torch

    import paper_2603_08661_amd as igsp

    dev = torch.device("cuda:0")
    W, H = (np.array(x, np.int32) for x in zip(*sizes))
    px = W.astype(np.int64) * H
    views = (W, H, np.r_[0, np.cumsum(3 * px)[:-1]], np.r_[0, np.cumsum(px)[:-1]])
    img = torch.randint(0, 256, (int(3 * px.sum()) + 16,), dtype=torch.uint8, device=dev)
    maps = [torch.zeros(int(px.sum()), device=dev) for _ in range(4)]
    torch.cuda.synchronize()
    held = {}
    for p, out in zip(("fp32", "bf16"), maps):
        igsp.edge_importance(img, views, out, precision=p, batched="staged")    # kernels loaded
    for p, out in zip(("fp32", "bf16"), maps):
        igsp.release_plans()
        free = torch.cuda.mem_get_info(dev)[0]
        igsp.edge_importance(img, views, out, precision=p, batched="staged")
        torch.cuda.synchronize()
        held[p] = free - torch.cuda.mem_get_info(dev)[0]
    bf16_map = int((-(-W // 248) * H.astype(np.int64)).sum()) * 512
    listed = 4 * int(px.sum()) // 16 if len(sizes) > 1 else 0
    extra = held["fp32"] - held["bf16"] - bf16_map - listed
    print(f"{extra / 2 ** 20:.1f} MiB besides", flush=True)
    assert extra < 5 * 2 ** 20
    # and both forms still give the same bits
    igsp.edge_importance(img, views, maps[1], precision="fp32", batched="plain")
    igsp.edge_importance(img, views, maps[2], precision="fp32", batched="unfused")
    torch.cuda.synchronize()
    assert torch.equal(maps[0], maps[1]) and torch.equal(maps[0], maps[2])
    igsp.release_plans()


def test_fp32_candidate_list_cut_off():
    """Two views of 712 chunks take the long chain together. One is striped with
    noise: every refinement work-group's list has room for what it finds (2048),
    but together they find more than the view's list holds (1/16 of its pixels), so
    the second pass reads the map; the other is textured and fits. Both equal the
    persistent form, which keeps no lists, bit for bit."""
    w, h, slots = 1984, 1424, 64
    rng = np.random.default_rng(23)
    noisy = np.zeros((h, w, 3)) + ((((np.arange(w) // 4) % 2) * 180) + 30)[None, :, None] + rng.normal(0, 1.0, (h, w, 1))
    noisy = np.clip(np.rint(noisy), 0, 255).astype(np.uint8)
    textured = synth.image(190, w, h, n_poly=20, texture=True)
    assert 8 * h // 16 == 712 and 2 * 8 * h < 40000          # long chain, 64 slots a work-group
    found = []
    for im in (noisy, textured):
        o = oracle.edge_view(im)
        med = np.float32(o["Mmed"]).view(np.uint32) >> 16
        hit = o["keep"].astype(bool) & (o["M"].astype(np.float32).view(np.uint32) >> 16 == med)
        found.append(hit.reshape(8 * h // slots, -1).sum(1))  # a work-group's slots: 8 strips of 8 rows
    assert found[0].max() <= 2048 and found[0].sum() > w * h // 16 >= found[1].sum(), [f.sum() for f in found]
    vb = synth.pack_views([noisy, textured], in_align=16, out_align=4)
    b, mb, nb = gpu_edge(vb, "fp32", "persistent")
    a, ma, na = gpu_edge(vb, "fp32", "staged", reps=3)
    assert np.array_equal(a, b) and np.array_equal(ma, mb) and np.array_equal(na, nb) and (na > 0).all()
