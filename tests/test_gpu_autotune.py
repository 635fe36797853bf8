"""Autotuning of the batched convolution's tile shapes (GPU): the maps are
bitwise the same for every segment height and workgroup count, and the tuned
plan gives the default plan's results."""
import ctypes

import pytest
import torch

from paper_1310_7114_amd import autotune as T
from paper_1310_7114_amd import synth as S

pytestmark = pytest.mark.gpu


def make_plan(itc, cases):
    plan = itc.BatchPlan([torch.from_numpy(c.img) for c in cases], [c.M for c in cases], [c.sigma for c in cases],
                         [c.iters for c in cases])
    return plan, plan.pack_codebooks([c.w0 for c in cases])


def maps_now(plan):
    plan.maps.zero_()
    plan.precompute()
    torch.cuda.synchronize()
    return plan.maps.clone()


def test_maps_do_not_depend_on_the_tile_shape(gpu_lib):
    cases = S.config3_cases(indices=range(0, 1400, 7))  # 200 silhouettes, every radius class
    plan, _ = make_plan(gpu_lib, cases)
    classes = plan.conv_classes()
    assert len(classes) == 3 and all(c["seg_rows"] == 256 for c in classes)
    ref = maps_now(plan)
    for seg, per in ((64, 0), (128, 1), (512, 0), (4096, 2), (192, 0)):
        for c in classes:
            plan.set_conv_shape(c["key"], seg, min(per, c["max_blocks_per_cu"]))
        assert torch.equal(maps_now(plan), ref), (seg, per)


def test_fp32_classes_take_earlier_shapes(gpu_lib):
    """FP32 weights of every radius: up to four workgroups a unit are accepted, and the maps stay the same."""
    radii = [2, 8, 12, 16, 24, 32]
    g = torch.Generator().manual_seed(5)
    imgs = [torch.rand((90 + 67 * i, 100 + 31 * i), generator=g) for i in range(6)]
    plan = gpu_lib.BatchPlan(imgs, [2] * 6, [r / 3 for r in radii], [1] * 6, radii=radii)
    classes = plan.conv_classes()
    assert [c["key"] for c in classes] == radii
    ref = maps_now(plan)
    for seg, per in ((64, 4), (128, 1), (512, 3), (256, 4)):
        for c in classes:
            plan.set_conv_shape(c["key"], seg, per)
        assert all(c["blocks_per_cu"] <= c["max_blocks_per_cu"] for c in plan.conv_classes())
        assert torch.equal(maps_now(plan), ref), (seg, per)


def test_tuned_plan_gives_the_default_results(gpu_lib, tmp_path):
    cases = S.config3_cases(indices=range(3, 1400, 14))
    plan, w0 = make_plan(gpu_lib, cases)
    n = plan.n

    def run():
        w = torch.empty_like(w0)
        sx = torch.empty(n, dtype=torch.float64, device="cuda")
        d = torch.empty_like(sx)
        done = torch.empty(n, dtype=torch.int32, device="cuda")
        plan.run(w0, w, sx, d, done)
        torch.cuda.synchronize()
        return w, sx, d

    ref = run()
    path = str(tmp_path / "tune.json")
    chosen = T.tune_conv(plan, reps=2, path=path)
    assert set(chosen) == {c["key"] for c in plan.conv_classes()}
    for key, ch in chosen.items():
        assert ch["seg_rows"] in T.SEG_CANDIDATES and not ch["cached"]
    for a, b in zip(run(), ref):
        assert torch.equal(a, b)
    # a second plan of the same layout takes the cached shapes
    plan2, _ = make_plan(gpu_lib, cases)
    again = T.tune_conv(plan2, reps=2, path=path)
    assert all(v["cached"] for v in again.values())
    assert {k: (v["seg_rows"], v["blocks_per_cu"]) for k, v in again.items()} == \
           {k: (v["seg_rows"], v["blocks_per_cu"]) for k, v in chosen.items()}


def test_graph_captured_after_tuning_replays_exactly(gpu_lib, tmp_path):
    """A graph captured after tuning equals eager execution on every replay
    (with eager work and synchronisation between the replays)."""
    cases = S.config3_cases(indices=range(5, 1400, 20))
    plan, w0 = make_plan(gpu_lib, cases)
    n = plan.n
    T.tune_conv(plan, reps=2, path=str(tmp_path / "tune.json"))
    w = torch.empty_like(w0)
    sx = torch.empty(n, dtype=torch.float64, device="cuda")
    d = torch.empty_like(sx)
    done = torch.empty(n, dtype=torch.int32, device="cuda")
    plan.run(w0, w, sx, d, done)
    torch.cuda.synchronize()
    ref = (w.clone(), sx.clone(), d.clone())
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        plan.run(w0, w, sx, d, done)
    torch.cuda.current_stream().wait_stream(side)
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        plan.run(w0, w, sx, d, done)
    for _ in range(3):
        w.zero_()
        d.zero_()
        torch.cuda.synchronize()
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(w, ref[0]) and torch.equal(sx, ref[1]) and torch.equal(d, ref[2])


def test_conv_launches_counts_every_kernel(gpu_lib):
    """The launch count of a plan is the number of kernels one `precompute` runs (read off a capture): one for a
    small plan, two a group where 320 MiB of weights are read ahead."""
    hip = ctypes.CDLL("libamdhip64.so")
    for plan in (gpu_lib.BatchPlan.for_stack(3, 200, 300, 1, 1.0, dtype=torch.uint8),
                 gpu_lib.BatchPlan.for_stack(3, 200, 301, 1, 1.0, dtype=torch.uint8),
                 gpu_lib.BatchPlan.for_stack(5, 8192, 8192, 1, 0.6, dtype=torch.uint8)):
        n = sum(h * w for h, w in plan.shapes)
        x = torch.zeros(n, dtype=torch.uint8, device="cuda")
        plan.precompute(weights=x)
        torch.cuda.synchronize()
        g = torch.cuda.CUDAGraph(keep_graph=True)
        with torch.cuda.graph(g):
            plan.precompute(weights=x)
        nodes = ctypes.c_size_t()
        assert hip.hipGraphGetNodes(ctypes.c_void_p(g.raw_cuda_graph()), None, ctypes.byref(nodes)) == 0
        assert plan.conv_launches() == nodes.value


MIB = 1 << 20


def stack_plan(itc, shapes, woffs=None, pitches=None):
    """A plan over uint8 images at the given byte offsets and pitches (a packed stack by default)."""
    n = len(shapes)
    return itc.BatchPlan(None, [1] * n, [0.6] * n, [0] * n, _shapes=shapes, _dtype=torch.uint8, _woffs=woffs,
                         _pitches=pitches)


def views(side, rows, cols, by_columns):
    """(shapes, offsets, pitches) of the rows x cols views that tile a side x side buffer."""
    at = [(u, v) for u in range(0, side, rows) for v in range(0, side, cols)]
    if by_columns:
        at.sort(key=lambda a: a[::-1])
    return [(rows, cols)] * len(at), [u * side + v for u, v in at], [side] * len(at)


READ_AHEAD = [
    # 256 MiB of weights in views whose rows are 16,384 bytes apart (with the gaps of every row they span 34 GB)
    ("views_256MiB", lambda: views(16384, 128, 128, False), 1),
    # 400 MiB: the views row by row fill whole bands of the buffer; column by column a group would read all of it
    ("views_by_rows", lambda: views(20480, 1024, 1024, False), 8),
    ("views_by_columns", lambda: views(20480, 1024, 1024, True), 1),
    # one image 300 times is one image's bytes
    ("one_image_300_times", lambda: ([(1024, 1024)] * 300, [0] * 300, [1024] * 300), 1),
    # above a group's size: not read ahead; small images beside one: three groups of at most 128 MiB, then the large one
    ("large_images", lambda: ([(12800, 12800)] * 2, None, None), 1),
    ("mixed", lambda: ([(6400, 6400)] * 4 + [(12800, 12800)] + [(6400, 6400)] * 4, None, None), 7),
    ("row_padding", lambda: ([(1000, 1000)] * 400, None, [1024] * 400), 6),  # 381 MiB without the padding
]


@pytest.mark.parametrize("name,build,launches", READ_AHEAD, ids=[c[0] for c in READ_AHEAD])
def test_read_ahead_groups(gpu_lib, name, build, launches):
    """Weights above 256 MiB are read ahead in groups of at most 128 MiB where a group's bytes are weights, not the
    gaps between the rows of views; the maps are those of the images alone, also after a change of the tile shape."""
    shapes, woffs, pitches = build()
    plan = stack_plan(gpu_lib, shapes, woffs, pitches)
    assert plan.conv_launches() == launches
    end = max(int(o) + (h - 1) * p + w for (h, w), o, p in zip(shapes, plan.weight_off, plan.pitches))
    g = torch.Generator(device="cuda").manual_seed(1)
    x = torch.randint(0, 256, (end,), generator=g, device="cuda", dtype=torch.uint8)
    some = sorted({0, len(shapes) // 3, len(shapes) - 1})

    for key in [None] + [c["key"] for c in plan.conv_classes()]:
        if key is not None:
            plan.set_conv_shape(key, 512, 1)
            assert plan.conv_launches() == launches
        plan.maps.zero_()
        plan.precompute(weights=x)
        for i in some:
            (h, w), p, o = shapes[i], plan.pitches[i], int(plan.weight_off[i])
            img = x[o: o + (h - 1) * p + w].as_strided((h, w), (p, 1))
            one = gpu_lib.precompute(img, 0.6)
            got = plan.maps_of(i)
            for a, b in zip(got.planes(), one.planes()):
                assert torch.equal(a, b)


def test_bad_shapes_are_rejected(gpu_lib):
    plan, _ = make_plan(gpu_lib, S.config3_cases(indices=range(4)))
    key = plan.conv_classes()[0]["key"]
    with pytest.raises(gpu_lib.ItcError):
        plan.set_conv_shape(key, 32, 0)
    with pytest.raises(gpu_lib.ItcError):
        plan.set_conv_shape(key, 8192, 0)
    with pytest.raises(gpu_lib.ItcError):
        plan.set_conv_shape(key, 256, 999)
    with pytest.raises(gpu_lib.ItcError):
        plan.set_conv_shape(12345, 256, 0)
