"""The march's candidate loop at the edges of its blocks: blocks of 64 list
entries, groups of four candidates, against the FP64 oracle."""
import numpy as np
import pytest

import oracle
from paper_2509_07782_amd import inputs

from helpers import oracle_opts, renderer_for

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch_cuda():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return torch


@pytest.mark.parametrize("n", [1, 2, 3, 4, 5, 7, 8, 63, 64, 65, 67, 128, 131])
def test_candidate_groups_against_oracle(torch_cuda, n):
    """n Gaussians that all cover the whole view: every segment's candidate
    list holds about n entries, so blocks and groups of every remainder run,
    forward, replaying backward and searching backward; brute force (blocks of
    consecutive Gaussians) gives the same bits."""
    torch = torch_cuda
    from paper_2509_07782_amd.render import RenderOptions
    rng = np.random.default_rng(400 + n)
    sc = inputs.make_scene("cluster", n, 41)
    sc["means"] = (0.05 * rng.standard_normal((n, 3))).astype(np.float32)
    sc["log_scales"] = rng.normal(-1.2, 0.3, (n, 3)).astype(np.float32)
    sc["density"] = (0.05 + rng.random(n)).astype(np.float32)
    cam = inputs.look_at_camera(19, 13, (0.1, 0.2, 2.5), fov_deg=20.0)
    r, p = renderer_for(sc)
    o = RenderOptions(dt=0.05, ess=1, t_eps=0.0)
    st = r.new_state()
    rgb, T = r.forward([cam], o, state=st)
    brute, Tb = r.forward([cam], RenderOptions(dt=0.05, ess=1, t_eps=0.0, brute_force=True))
    assert torch.equal(rgb, brute) and torch.equal(T, Tb)
    oo = oracle_opts(o)
    orgb, oT, _, _ = oracle.render(sc, cam, oo)
    # FP32 sums of n terms of order one
    assert np.abs(rgb.cpu().numpy() - orgb).max() <= 1e-4
    assert np.abs(T.cpu().numpy() - oT).max() <= 1e-4
    g = np.random.default_rng(7).standard_normal(orgb.shape)
    gt = torch.from_numpy(g.astype(np.float32)).cuda()
    ref = oracle.backward(sc, cam, oo, np.arange(cam.n_rays), g, np.zeros(cam.n_rays))
    for state_opts in (o, RenderOptions(dt=0.05, ess=1, t_eps=0.0, no_record=True)):
        s2 = r.new_state()
        rgb2, T2 = r.forward([cam], state_opts, state=s2)
        grads = r.backward(s2, rgb2, T2, gt, None, p)
        for k, v in grads.items():
            a = v.cpu().numpy().astype(np.float64)
            assert np.linalg.norm(a - ref[k]) <= 1e-3 * max(np.linalg.norm(ref[k]), 1e-30), (k, n)
    r.check_errors()


@pytest.mark.parametrize("kind,n,sd,eye,fov,tile", [
    ("cluster", 3, 0.5, (0.0, 0.1, 2.0), 50.0, (8, 8)),          # absent children
    ("cluster", 20_000, 0.5, (0.05, 0.1, 0.2), 60.0, (8, 8)),     # camera inside ellipsoids
    ("cluster", 20_000, 0.5, (0.0, 0.1, 2.5), 160.0, (64, 1)),    # packets wider than the cone test
    ("outdoor", 30_000, 1.0, (0.3, 0.0, 0.4), 60.0, (8, 8)),      # anisotropic, large and far boxes
    ("outdoor", 30_000, 1.0, (0.3, 0.0, 0.4), 160.0, (16, 4)),
])
def test_collection_finds_every_hit(torch_cuda, kind, n, sd, eye, fov, tile):
    """The window collection against brute force, bit for bit: a Gaussian that
    a box or support test wrongly drops would change a pixel."""
    torch = torch_cuda
    from paper_2509_07782_amd.render import RenderOptions
    sc = inputs.make_scene(kind, n, 77, log_scale_sd=sd)
    far = 128.0 if kind == "outdoor" else 6.0
    cam = inputs.look_at_camera(53, 37, eye, target=(0.0, 0.05, 0.0), fov_deg=fov, t_far=far)
    r, _ = renderer_for(sc)
    kw = dict(adaptive=True, ess=1, t_eps=1e-4, tile_w=tile[0], tile_h=tile[1])
    rgb, T = r.forward([cam], RenderOptions(**kw))
    brute, Tb = r.forward([cam], RenderOptions(brute_force=True, **kw))
    assert torch.equal(rgb, brute) and torch.equal(T, Tb)
    r.check_errors()


@pytest.mark.parametrize("kind,n,eye,size,views,n_s,n_sg", [
    ("cluster", 3_000, (0.0, 0.2, 2.6), (67, 45), 1, 8, 0),       # 4 lanes a ray, ragged
    ("cluster", 3_000, (0.0, 0.2, 2.6), (67, 45), 1, 4, 0),
    ("cluster", 3_000, (0.0, 0.2, 2.6), (61, 37), 2, 16, 0),
    ("cluster", 3_000, (0.0, 0.2, 2.6), (45, 39), 1, 8, 7),
    ("cluster", 20_000, (0.0, 0.2, 2.6), (163, 129), 1, 8, 0),    # over one tile per CU
    ("cluster", 20_000, (0.1, 0.2, 0.1), (163, 129), 1, 8, 0),    # camera inside: one lane a ray
    ("cluster", 20_000, None, (163, 129), 2, 8, 0),               # one view inside, one outside
    ("cluster", 30_000, (0.0, 0.2, 2.6), (253, 249), 1, 8, 0),    # 2 lanes a ray
    ("cluster", 30_000, None, (179, 177), 2, 4, 0),
    ("cluster", 30_000, (0.0, 0.2, 2.6), (253, 249), 1, 16, 0),
])
@pytest.mark.parametrize("fixed,persistent", [(False, False), (True, True)])
def test_lanes_per_ray_give_the_same_rays(torch_cuda, kind, n, eye, size, views, n_s, n_sg, fixed,
                                          persistent):
    """A call that asks for statistics marches one lane per ray; without them
    small calls share a ray between 2 or 4 lanes.  Same images bit for bit;
    the gradients (replayed, and searched again) differ by the order of the
    FP32 sums over rays alone."""
    torch = torch_cuda
    from paper_2509_07782_amd.render import RenderOptions, Renderer
    sc = inputs.make_scene(kind, n, 91, sh_degree=2 if n_sg else None, n_sg=n_sg)
    keys = ("means", "log_scales", "quats", "density", "sh") + (("sg",) if n_sg else ())
    p = {k: torch.from_numpy(sc[k]).cuda() for k in keys}
    r = Renderer(0)
    r.build(p, sc["sh_degree"])
    eyes = [eye] * views if eye is not None else [(0.1, 0.2, 0.1), (0.0, 0.2, 2.6)]
    cams = [inputs.look_at_camera(*size, e, target=(0.0, 0.1 * i, -0.1)) for i, e in enumerate(eyes)]
    kw = dict(adaptive=not fixed, dt=0.01, n_s=n_s, ess=1, t_eps=1e-4, persistent=persistent)
    o = RenderOptions(**kw)
    one, many, own = r.new_state(), r.new_state(), r.new_state()
    rgb, T, _ = r.forward(cams, o, stats=True, state=one)
    rgb2, T2 = r.forward(cams, o, state=many)
    assert torch.equal(rgb, rgb2) and torch.equal(T, T2)
    g = torch.from_numpy(np.random.default_rng(3).standard_normal(tuple(rgb.shape)).astype(np.float32)).cuda()
    ref = r.backward(one, rgb, T, g, None, p)
    r.forward(cams, RenderOptions(no_record=True, **kw), state=own)
    for st in (many, own):
        grads = r.backward(st, rgb, T, g, None, p)
        for k in keys:
            a, b = grads[k].double(), ref[k].double()
            assert float((a - b).norm()) <= 2e-5 * float(b.norm()), k
    r.check_errors()
    r.close()


def test_densify_views_of_two_launches(torch_cuda):
    """26 views fill one launch (24) and start a second; every view's statistic
    equals that of a call of its own (FP32 sums over rays in another order)."""
    torch = torch_cuda
    from paper_2509_07782_amd.render import RenderOptions
    n, views = 700, 26
    sc = inputs.make_scene("cluster", n, 5)
    r, p = renderer_for(sc)
    cams = [inputs.look_at_camera(19, 13, (2.5 * np.sin(v), 0.1 * v - 1.0, 2.5 * np.cos(v)))
            for v in range(views)]
    o = RenderOptions(adaptive=True, ess=1, t_eps=1e-4)
    rng = np.random.default_rng(6)

    def statistic(group, g):
        st = r.new_state()
        rgb, T = r.forward(group, o, state=st)
        stat = torch.zeros(n, device="cuda")
        seen = torch.zeros(n, device="cuda", dtype=torch.int32)
        grads = r.backward(st, rgb, T, g, None, p, stat, seen)
        return stat.double(), seen, grads["means"].double()

    g = torch.from_numpy(rng.standard_normal((views * 247, 3)).astype(np.float32)).cuda()
    stat, seen, gm = statistic(cams, g)
    one = [statistic([c], g[247 * v:247 * (v + 1)].contiguous()) for v, c in enumerate(cams)]
    ref, ref_gm = sum(x[0] for x in one), sum(x[2] for x in one)
    assert float((stat - ref).norm()) <= 2e-5 * float(ref.norm())
    assert float((gm - ref_gm).norm()) <= 2e-5 * float(ref_gm.norm())
    assert torch.equal(seen, sum(x[1] for x in one))
    r.check_errors()


def test_densify_captured_after_fewer_views(torch_cuda):
    """A capture of three views after an eager call of one: the views' buffer
    cannot grow there and holds one view at a time; every replay gives what
    the eager call gives."""
    torch = torch_cuda
    from paper_2509_07782_amd.render import RenderOptions
    n = 700
    sc = inputs.make_scene("cluster", n, 23)
    cams = [inputs.look_at_camera(21, 17, (x, 0.4, 2.2), fov_deg=45.0) for x in (-0.6, 0.1, 0.7)]
    r, p = renderer_for(sc)
    o = RenderOptions(dt=0.02, ess=1)
    stat = torch.zeros(n, device="cuda")
    seen = torch.zeros(n, dtype=torch.int32, device="cuda")
    gt = torch.from_numpy(np.random.default_rng(3).standard_normal((3 * 21 * 17, 3))
                          .astype(np.float32)).cuda()
    s1 = r.new_state()
    rgb, T = r.forward(cams[:1], o, state=s1)
    r.backward(s1, rgb, T, gt[:21 * 17].contiguous(), None, p, densify=stat, densify_views=seen)
    s3 = r.new_state()
    rgb, T = r.forward(cams, o, state=s3)
    r.backward(s3, rgb, T, gt, None, p)   # (the launches, without the statistic)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        captured = r.backward(s3, rgb, T, gt, None, p, densify=stat, densify_views=seen)
    got = []
    for _ in range(3):
        stat.zero_()
        seen.zero_()
        graph.replay()
        torch.cuda.synchronize()
        got.append((stat.clone(), seen.clone(), {k: v.clone() for k, v in captured.items()}))
    stat.zero_()
    seen.zero_()
    eager = r.backward(s3, rgb, T, gt, None, p, densify=stat, densify_views=seen)
    torch.cuda.synchronize()
    assert int(seen.sum()) > 0
    for st, se, gr in got:
        assert torch.equal(se, seen)
        # the order of the atomic sums differs, a few rounding errors of each
        assert float((st - stat).norm()) <= 1e-4 * float(stat.norm())
        for k, v in eager.items():
            assert float((gr[k] - v).norm()) <= 1e-4 * float(v.norm()), k
    r.check_errors()


def test_densify_capture_outlives_larger_calls(torch_cuda):
    """A captured one-view densification backward, an eager call of three
    views (the views' buffer grows), new allocations, then replays: the graph
    still owns the memory it addresses and gives what its eager call gave."""
    torch = torch_cuda
    from paper_2509_07782_amd.render import RenderOptions
    n, px = 700, 21 * 17
    sc = inputs.make_scene("cluster", n, 23)
    cams = [inputs.look_at_camera(21, 17, (x, 0.4, 2.2), fov_deg=45.0) for x in (-0.6, 0.1, 0.7)]
    r, p = renderer_for(sc)
    o = RenderOptions(dt=0.02, ess=1)
    gt = torch.from_numpy(np.random.default_rng(3).standard_normal((3 * px, 3)).astype(np.float32)).cuda()
    g1 = gt[:px].contiguous()

    def buffers():
        return torch.zeros(n, device="cuda"), torch.zeros(n, dtype=torch.int32, device="cuda")

    stat, seen = buffers()
    s1, s3 = r.new_state(), r.new_state()
    rgb, T = r.forward(cams[:1], o, state=s1)
    eager = r.backward(s1, rgb, T, g1, None, p, densify=stat, densify_views=seen)
    ref_stat, ref_seen = stat.clone(), seen.clone()
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        captured = r.backward(s1, rgb, T, g1, None, p, densify=stat, densify_views=seen)
    rgb3, T3 = r.forward(cams, o, state=s3)
    stat3, seen3 = buffers()
    r.backward(s3, rgb3, T3, gt, None, p, densify=stat3, densify_views=seen3)
    others = [torch.full((n * k,), float("nan"), device="cuda") for k in (3, 6, 9)]
    for _ in range(2):
        stat.zero_()
        seen.zero_()
        graph.replay()
        torch.cuda.synchronize()
        assert int(seen.sum()) > 0 and torch.equal(seen, ref_seen)
        # the order of the atomic sums differs, a few rounding errors of each
        assert float((stat - ref_stat).norm()) <= 1e-4 * float(ref_stat.norm())
        for k, v in eager.items():
            assert float((captured[k] - v).norm()) <= 1e-4 * float(v.norm()), k
        assert all(bool(t.isnan().all()) for t in others)
    r.check_errors()


@pytest.mark.parametrize("size,tile,n", [
    ((1, 140_000), (8, 8), 120_000),    # 35000 rows of tiles, 4 lanes a ray
    ((1, 270_000), (8, 8), 120_000),    # 67500, 2 lanes: no tile table
    ((2, 262_200), (8, 8), 3_000),      # 32775, one lane
    ((70_003, 2), (1, 64), 3_000),      # 70003 columns, 2 lanes: no tile table
])
def test_long_thin_images(torch_cuda, size, tile, n):
    """Images with more tiles on a side than a signed or unsigned 16-bit
    number counts: every pixel, and the gradients, as with rays in row order
    (which has no tiles)."""
    torch = torch_cuda
    from paper_2509_07782_amd.render import RenderOptions
    sc = inputs.make_scene("cluster", n, 19)
    w, h = size
    pose = inputs.look_at_camera(8, 8, (0.2, 0.1, 2.6)).cam_to_world
    f = 0.9 * max(w, h)
    cam = inputs.Camera(w, h, f, f, w / 2.0, h / 2.0, pose, 0.0, 6.0)
    r, p = renderer_for(sc)
    kw = dict(adaptive=True, ess=1, t_eps=1e-4)
    o = RenderOptions(tile_w=tile[0], tile_h=tile[1], **kw)
    st, own = r.new_state(), r.new_state()
    rgb, T = r.forward([cam], o, state=st)
    ref, ref_T = r.forward([cam], RenderOptions(ray_order=0, **kw), state=own)
    assert torch.equal(rgb, ref) and torch.equal(T, ref_T)
    assert float((1 - T).max()) > 0.1
    g = torch.from_numpy(np.random.default_rng(2).standard_normal(tuple(rgb.shape)).astype(np.float32)).cuda()
    a, b = r.backward(st, rgb, T, g, None, p), r.backward(own, ref, ref_T, g, None, p)
    for k, v in b.items():
        # the same terms in another order of the atomic sums
        assert float((a[k] - v).norm()) <= 2e-5 * float(v.norm()), k
    r.check_errors()


@pytest.mark.parametrize("warm", ["more views", "statistics"])
def test_capture_after_calls_with_one_lane_a_ray(torch_cuda, warm):
    """A small forward and its backward captured after eager calls whose rays
    had one lane each: nothing is left to allocate, and every replay gives the
    eager result."""
    torch = torch_cuda
    from paper_2509_07782_amd.render import RenderOptions
    sc = inputs.make_scene("cluster", 3_000, 29)
    cams = [inputs.look_at_camera(163, 129, (2.5 * np.sin(v), 0.3, 2.5 * np.cos(v))) for v in range(8)]
    r, p = renderer_for(sc)
    o = RenderOptions(adaptive=True, ess=1, t_eps=1e-4)
    st, ref = r.new_state(), r.new_state()
    g = torch.from_numpy(np.random.default_rng(4).standard_normal((163 * 129, 3)).astype(np.float32)).cuda()
    if warm == "more views":
        rgb, T = r.forward(cams, o, state=st)
        r.backward(st, rgb, T, g.repeat(8, 1), None, p)
    else:
        rgb, T, _ = r.forward(cams[:1], o, stats=True, state=st)
        r.backward(st, rgb, T, g, None, p)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        rgb, T = r.forward(cams[:1], o, state=st)
        got = r.backward(st, rgb, T, g, None, p)
    eager, eager_T = r.forward(cams[:1], o, state=ref)
    want = r.backward(ref, eager, eager_T, g, None, p)
    for _ in range(3):
        rgb.zero_()
        T.zero_()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(rgb, eager) and torch.equal(T, eager_T)
        for k, v in want.items():
            # the order of the sums over rays differs
            assert float((got[k] - v).norm()) <= 2e-5 * float(v.norm()), k
    r.check_errors()


def test_capture_after_calls_with_shared_rays(torch_cuda):
    """Eight views captured after an eager call of one, whose rays were shared
    between lanes: the tables of their 64-ray tiles are there."""
    torch = torch_cuda
    from paper_2509_07782_amd.render import RenderOptions
    sc = inputs.make_scene("cluster", 3_000, 29)
    cams = [inputs.look_at_camera(163, 129, (2.5 * np.sin(v), 0.3, 2.5 * np.cos(v))) for v in range(8)]
    r, _ = renderer_for(sc)
    o = RenderOptions(adaptive=True, ess=1, t_eps=1e-4)
    r.forward(cams[:1], o)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        rgb, T = r.forward(cams, o)
    eager, eager_T = r.forward(cams, o)
    for _ in range(3):
        rgb.zero_()
        T.zero_()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(rgb, eager) and torch.equal(T, eager_T)
    r.check_errors()


@pytest.mark.parametrize("size,fov,tile", [((53, 37), 60.0, (8, 8)), ((53, 37), 160.0, (64, 1)),
                                           ((320, 213), 60.0, (8, 8)), ((320, 213), 160.0, (64, 1))])
@pytest.mark.parametrize("scales", [(45.0, 45.0, 45.0), (45.0, -3.0, -3.0), (43.0, 43.0, -2.0)])
def test_boxes_with_infinite_sides(torch_cuda, size, fov, tile, scales):
    """A Gaussian whose box overflows to infinite sides makes every node above
    it infinite: nothing below them is lost (brute force, bit for bit).  Narrow
    packets and ones too wide for the cone test, one and four lanes a ray."""
    torch = torch_cuda
    from paper_2509_07782_amd.render import RenderOptions
    sc = inputs.make_scene("cluster", 2_000, 31)
    for i in (5, 900):
        sc["log_scales"][i] = np.float32(scales)
        sc["density"][i] = 0.5
    cam = inputs.look_at_camera(*size, (0.0, 0.1, 2.4), fov_deg=fov)
    r, _ = renderer_for(sc)
    kw = dict(adaptive=True, ess=1, t_eps=1e-4, tile_w=tile[0], tile_h=tile[1])
    rgb, T = r.forward([cam], RenderOptions(**kw))
    one, one_T, _ = r.forward([cam], RenderOptions(**kw), stats=True)
    brute, brute_T = r.forward([cam], RenderOptions(brute_force=True, **kw))
    assert float((1 - brute_T).max()) > 0.5
    assert torch.equal(rgb, brute) and torch.equal(T, brute_T)
    assert torch.equal(one, brute) and torch.equal(one_T, brute_T)
    r.check_errors()


@pytest.mark.parametrize("n,eye,size,views,n_s,n_sg", [
    (3_000, (0.0, 0.2, 2.6), (67, 45), 1, 8, 0),          # 4 lanes a ray
    (3_000, (0.0, 0.2, 2.6), (61, 37), 2, 16, 0),
    (3_000, (0.0, 0.2, 2.6), (45, 39), 1, 8, 7),
    (30_000, (0.0, 0.2, 2.6), (253, 249), 1, 8, 0),       # 2 lanes
    (20_000, None, (163, 129), 2, 8, 0),                  # one view inside, one outside
    (3_000, (0.0, 0.2, 2.6), (403, 301), 1, 8, 0),        # one lane
])
@pytest.mark.parametrize("persistent", [False, True])
def test_partly_recorded_forwards(torch_cuda, n, eye, size, views, n_s, n_sg, persistent):
    """Record pools from 4 MB to 16 KB: from a few tiles without a record to a
    few with one.  Images are unchanged, and the gradients are those of a
    backward that searches every tile itself."""
    torch = torch_cuda
    from paper_2509_07782_amd.render import RenderOptions, Renderer
    sc = inputs.make_scene("cluster", n, 91, sh_degree=2 if n_sg else None, n_sg=n_sg)
    keys = ("means", "log_scales", "quats", "density", "sh") + (("sg",) if n_sg else ())
    p = {k: torch.from_numpy(sc[k]).cuda() for k in keys}
    r = Renderer(0)
    r.build(p, sc["sh_degree"])
    eyes = [eye] * views if eye is not None else [(0.1, 0.2, 0.1), (0.0, 0.2, 2.6)]
    cams = [inputs.look_at_camera(*size, e, target=(0.0, 0.1 * i, -0.1)) for i, e in enumerate(eyes)]
    kw = dict(adaptive=True, n_s=n_s, ess=1, t_eps=1e-4, persistent=persistent)
    own, st = r.new_state(), r.new_state()
    rgb, T = r.forward(cams, RenderOptions(no_record=True, **kw), state=own)
    g = torch.from_numpy(np.random.default_rng(3).standard_normal(tuple(rgb.shape)).astype(np.float32)).cuda()
    ref = r.backward(own, rgb, T, g, None, p)
    for limit in (1 << 22, 1 << 20, 1 << 18, 1 << 16, 1 << 14):
        r.ctx.set_record_limit(limit)
        for lean in (False, True):
            rgb2, T2 = r.forward(cams, RenderOptions(no_sample_record=lean, **kw), state=st)
            assert torch.equal(rgb, rgb2) and torch.equal(T, T2)
            grads = r.backward(st, rgb, T, g, None, p)
            assert r.ctx.backward_replayed()
            for k in keys:
                # the same terms in another order of the FP32 sums
                assert float((grads[k] - ref[k]).norm()) <= 2e-5 * float(ref[k].norm()), (k, limit, lean)
    r.check_errors()
    r.close()


@pytest.mark.parametrize("limit", [0, 1 << 20])
def test_chunked_windows_of_shared_rays(torch_cuda, limit):
    """Dense lists that come in several chunks, with 4 and 2 lanes a ray: the
    replay reads the chunks again as it does with one lane."""
    torch = torch_cuda
    from paper_2509_07782_amd.render import RenderOptions
    sc = inputs.make_scene("cluster", 40_000, 33)
    sc["log_scales"] += np.float32(0.7)
    r, p = renderer_for(sc)
    r.ctx.set_record_limit(limit)
    for size in ((96, 72), (253, 249)):
        cam = inputs.look_at_camera(*size, (0.9, 0.3, 2.2), fov_deg=50.0)
        kw = dict(adaptive=True, ess=1, t_eps=1e-4, window_segments=4)
        st, own = r.new_state(), r.new_state()
        ref, ref_T, stats = r.forward([cam], RenderOptions(no_record=True, **kw), stats=True, state=own)
        assert own.totals()["chunked"] > 0
        rgb, T = r.forward([cam], RenderOptions(**kw), state=st)
        assert torch.equal(rgb, ref) and torch.equal(T, ref_T)
        g = torch.from_numpy(np.random.default_rng(5).standard_normal(tuple(rgb.shape)).astype(np.float32)).cuda()
        a, b = r.backward(st, rgb, T, g, None, p), r.backward(own, ref, ref_T, g, None, p)
        for k, v in b.items():
            assert float((a[k] - v).norm()) <= 2e-5 * float(v.norm()), (k, size)
    r.check_errors()


@pytest.mark.parametrize("limit,whole", [(0, True), (1 << 22, False)])
def test_records_of_one_tile_in_many_shares(torch_cuda, limit, whole):
    """One tile whose records (several MB) fill one share of the pool after
    another: recorded whole in the default pool, not in a smaller one, and the
    gradients are those of a backward that searches."""
    torch = torch_cuda
    from paper_2509_07782_amd.render import RenderOptions
    sc = inputs.make_scene("cluster", 20_000, 37)
    cam = inputs.look_at_camera(8, 8, (0.2, 0.1, 2.4), fov_deg=30.0)
    r, p = renderer_for(sc)
    r.ctx.set_record_limit(limit)
    kw = dict(dt=0.0005, ess=1, t_eps=0.0)
    st, own = r.new_state(), r.new_state()
    ref, ref_T = r.forward([cam], RenderOptions(no_record=True, **kw), state=own)
    rgb, T, _ = r.forward([cam], RenderOptions(**kw), stats=True, state=st)
    assert st.totals()["unrecorded"] == (0 if whole else 1)
    assert torch.equal(rgb, ref) and torch.equal(T, ref_T)
    g = torch.from_numpy(np.random.default_rng(6).standard_normal((64, 3)).astype(np.float32)).cuda()
    a, b = r.backward(st, rgb, T, g, None, p), r.backward(own, ref, ref_T, g, None, p)
    for k, v in b.items():
        assert float((a[k] - v).norm()) <= 2e-5 * float(v.norm()), k
    r.check_errors()
