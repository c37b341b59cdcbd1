"""CPU-only tests of the HIP library's host side: it loads, exports what
include/sfc.h declares, validates arguments without touching a GPU, and its add
networks (compiled for the host) realize the oracle's matrices."""
import ctypes as C
import os
import re
import struct
import subprocess

import numpy as np
import pytest

from oracle import sfc as oracle

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HEADER = os.path.join(ROOT, "include", "sfc.h")


@pytest.fixture(scope="module")
def lib():
    from paper_2407_02913_amd import binding

    if not os.path.exists(binding.LIB_PATH):
        import __graft_entry__ as entry

        entry.build()
    return binding.load()


def declared_functions():
    text = open(HEADER).read()
    text = re.sub(r"/\*.*?\*/", "", text, flags=re.S)
    return sorted(set(re.findall(r"\b(sfc_[a-z0-9_]+)\s*\(", text)))


def test_header_declares_the_three_named_entry_points():
    names = declared_functions()
    for must in ("sfc_plan", "sfc_transform_filter", "sfc_conv2d_nchw"):
        assert must in names


def test_library_exports_every_declared_symbol(lib):
    from paper_2407_02913_amd import binding

    names = declared_functions()
    assert sorted(binding.EXPORTS) == names
    for n in names:
        assert hasattr(lib, n), n


def test_missing_library_fails_loudly(monkeypatch, tmp_path):
    from paper_2407_02913_amd import binding

    monkeypatch.setattr(binding, "LIB_PATH", str(tmp_path / "nope.so"))
    monkeypatch.setattr(binding, "_lib", None)
    with pytest.raises(RuntimeError, match="no CPU fallback"):
        binding.load()


@pytest.mark.parametrize("missing", [(), ("_cuda_getCurrentRawStream",), ("_cuda_getDevice",)])
def test_current_stream_with_and_without_the_raw_handle(monkeypatch, missing):
    """The handle of the current device's current stream, from torch's undocumented names where
    it has them, else from the Stream object."""
    from types import SimpleNamespace

    import torch

    from paper_2407_02913_amd import binding

    monkeypatch.setattr(binding, "_raw_stream", None)
    monkeypatch.setattr(binding, "_device", None)
    monkeypatch.setattr(torch._C, "_cuda_getCurrentRawStream", lambda d: 1000 + d, raising=False)
    monkeypatch.setattr(torch._C, "_cuda_getDevice", lambda: 3, raising=False)
    monkeypatch.setattr(torch.cuda, "current_device", lambda: 3)
    monkeypatch.setattr(torch.cuda, "current_stream", lambda d=None: SimpleNamespace(cuda_stream=2000 + d))
    for name in missing:
        monkeypatch.delattr(torch._C, name)
    want = 2003 if missing else 1003
    assert [binding._stream_ptr(None) for _ in range(2)] == [want, want]
    assert binding._stream_ptr(SimpleNamespace(cuda_stream=5)) == 5


def make_desc(**kw):
    from paper_2407_02913_amd import binding

    base = dict(N=2, Cin=16, Cout=24, H=14, W=9, alg=0, mode=1, out=0, path=0, per_channel_wscale=1,
                transform_bits=0, flags=0)
    base.update(kw)
    return binding.ConvDesc(**base)


def plan_status(lib, desc):
    h = C.c_void_p()
    st = lib.sfc_plan(C.byref(desc), C.byref(h))
    return st, h


def test_plan_sizes_and_counts(lib):
    st, h = plan_status(lib, make_desc())
    assert st == 0
    fb, wb, p, t = C.c_size_t(), C.c_size_t(), C.c_int32(), C.c_int64()
    assert lib.sfc_plan_sizes(h, C.byref(fb), C.byref(wb), C.byref(p), C.byref(t)) == 0
    th, tw = oracle.tile_grid(14, 9)
    assert p.value == oracle.multiplications_per_tile("6x6_p88") == 88
    assert t.value == 2 * th * tw
    tp, cp, kp = -(-t.value // 16) * 16, 64, 32
    assert fb.value >= 88 * kp * cp + 2 * 88 * kp * 4
    assert wb.value >= 88 * tp * cp + 88 * tp * kp * 4
    assert lib.sfc_plan_sizes(h, None, None, None, None) == 0
    lib.sfc_plan_destroy(h)
    st, h = plan_status(lib, make_desc(alg=1, mode=0))
    assert st == 0
    assert lib.sfc_plan_sizes(h, C.byref(fb), C.byref(wb), C.byref(p), C.byref(t)) == 0
    assert p.value == 100 and fb.value >= 100 * kp * cp * 2
    lib.sfc_plan_destroy(h)


@pytest.mark.parametrize(
    "kw,code",
    [
        (dict(N=0), 1), (dict(Cin=-1), 1), (dict(H=0), 1), (dict(alg=10), 1), (dict(alg=-2), 1),
        (dict(mode=2), 1), (dict(out=5), 1), (dict(path=3), 1), (dict(path=-2), 1),
        (dict(per_channel_wscale=2), 1), (dict(flags=2), 1),
        (dict(transform_bits=1), 1), (dict(transform_bits=9), 1),
        (dict(transform_bits=4, mode=0), 2),  # exact mode has no transform-domain rounding
        (dict(out=1, mode=1), 2),  # raw integer output only in exact mode
        (dict(path=1, mode=0), 2),  # fused path is the requantized one
        (dict(W=5000), 2),
        # exact mode keeps 32-bit sums: guaranteed up to 404 channels (3x3), 145 (5x5 filters),
        # 74 (7x7 filters)
        (dict(mode=0, Cin=405), 2), (dict(mode=0, alg=6, Cin=146), 2), (dict(mode=0, alg=8, Cin=75), 2),
        (dict(Cout=65521), 2),  # one workgroup row per (padded) filter must fit a launch grid
    ],
)
def test_plan_rejects_bad_descriptions(lib, kw, code):
    st, h = plan_status(lib, make_desc(**kw))
    assert st == code and not h.value


def test_exact_mode_channel_bound_and_its_opt_in(lib):
    for kw in (dict(mode=0, Cin=404), dict(mode=0, alg=6, Cin=145), dict(mode=0, alg=9, Cin=74),
               dict(mode=0, Cin=512, flags=1),
               dict(mode=1, Cin=512)):
        st, h = plan_status(lib, make_desc(**kw))
        assert st == 0, kw
        lib.sfc_plan_destroy(h)


def test_auto_algorithm_and_path(lib):
    """SFC_ALG_AUTO / SFC_PATH_AUTO: the library's choice per layer shape, reported by
    sfc_plan_choice; an explicit choice is kept.  The ResNet shapes and the 13-layer stack get
    what bench.py runs (it asks for auto and reads the choice back)."""
    from paper_2407_02913_amd import binding, synth

    def choice(shape, **kw):
        plan = binding.Plan(shape.N, shape.Cin, shape.Cout, shape.H, shape.W, **kw)
        got = (plan.alg, plan.path)
        plan.close()
        return got

    want = {"tiny32": ("4x4_p46", "single"), "resnet56": ("4x4_p46", "single"),
            "resnet28": ("4x4_p46", "single"), "resnet14": ("4x4_p46", "fused"),
            "resnet7": ("7x7_p132", "staged"), "cifar16": ("4x4_p46", "single"),
            "cifar8": ("4x4_p46", "fused")}
    for name, shape in synth.LAYERS.items():
        assert choice(shape, alg="auto", path="auto") == want[name], name
    assert choice(synth.LAYERS["resnet56"], alg="6x6_p88", path="staged") == ("6x6_p88", "staged")
    assert choice(synth.LAYERS["resnet56"], alg="7x7_p132", path="auto") == ("7x7_p132", "single")
    # 512 channels on 7x7 maps: one 7x7 tile per image through the batched GEMMs from batch 128 on
    r7 = synth.LAYERS["resnet7"]
    assert choice(synth.LayerShape("b128", 128, r7.Cin, r7.Cout, 7, 7, "relu", True, 9), alg="auto",
                  path="auto") == ("7x7_p132", "staged")
    assert choice(synth.LayerShape("b64", 64, r7.Cin, r7.Cout, 7, 7, "relu", True, 9), alg="auto",
                  path="auto") == ("4x4_p46", "fused")
    # exact mode runs staged, on the 6x6 form the paper's headline count is about
    assert choice(synth.LAYERS["tiny32"], alg="auto", path="auto", mode="exact") == ("6x6_p88", "staged")
    # channel counts the fused kernel does not take (three 64-channel slices) fall back
    odd = synth.LayerShape("odd", 2, 192, 32, 14, 14, "relu", True, 9)
    assert choice(odd, alg="auto", path="auto")[1] == "staged"
    for shape in synth.stack_layers():
        alg, path = choice(shape, alg="auto", path="auto", out="i8")
        assert alg == binding.AUTO_ALG_3X3
        assert path == ("single" if shape.Cin <= binding.SINGLE_MAX_CIN else "fused")


def test_undersized_buffers_are_refused_before_any_launch(lib):
    """Every call that takes a caller-owned device buffer takes its size and returns
    SFC_EWORKSPACE when it is too small (no GPU here: a launch would fail differently)."""
    st, h = plan_status(lib, make_desc())
    assert st == 0
    fb, wb = C.c_size_t(), C.c_size_t()
    assert lib.sfc_plan_sizes(h, C.byref(fb), C.byref(wb), None, None) == 0
    p = 88
    sx = (C.c_float * p)(*([0.5] * p))
    sw = (C.c_float * (p * 24))(*([0.25] * (p * 24)))
    assert lib.sfc_set_point_scales(h, sx, sw) == 0
    ws = (C.c_float * 24)(*([0.01] * 24))
    dev = C.c_void_p(4096)
    assert lib.sfc_transform_filter(h, dev, ws, dev, fb.value - 1, None) == 6
    assert lib.sfc_conv2d_nchw(h, dev, C.c_float(1.0), dev, dev, wb.value - 1, None) == 6
    assert lib.sfc_conv2d_stages(h, dev, C.c_float(1.0), dev, dev, 0, None, 7) == 6
    out = (C.c_float * (p * 24))()
    assert lib.sfc_calibrate_act_scales(h, dev, 1, dev, wb.value - 1, None, out) == 6
    assert lib.sfc_calibrate_filter_scales(h, dev, dev, wb.value - 1, None, out) == 6
    # large enough: the next check in line answers (the filter has not been transformed)
    assert lib.sfc_conv2d_nchw(h, dev, C.c_float(1.0), dev, dev, wb.value, None) == 4
    assert lib.sfc_status_string(6) == b"device buffer smaller than the plan needs"
    lib.sfc_plan_destroy(h)


def test_null_and_order_errors_without_gpu(lib):
    assert lib.sfc_plan(None, None) == 1
    st, h = plan_status(lib, make_desc())
    assert st == 0
    p = 88
    sx = (C.c_float * p)(*([0.5] * p))
    sw = (C.c_float * (p * 24))(*([0.25] * (p * 24)))
    assert lib.sfc_set_point_scales(h, None, sw) == 1
    bad = (C.c_float * p)(*([0.5] * (p - 1) + [0.0]))
    assert lib.sfc_set_point_scales(h, bad, sw) == 1
    nan = (C.c_float * p)(*([0.5] * (p - 1) + [float("nan")]))
    assert lib.sfc_set_point_scales(h, nan, sw) == 1
    assert lib.sfc_set_point_scales(h, sx, sw) == 0
    # conv before the filter transform, and misaligned / null pointers: rejected before any launch
    big = C.c_size_t(1 << 40)
    assert lib.sfc_conv2d_nchw(h, C.c_void_p(256), C.c_float(1.0), C.c_void_p(512), C.c_void_p(1024), big, None) == 4
    assert lib.sfc_conv2d_nchw(h, None, C.c_float(1.0), C.c_void_p(512), C.c_void_p(1024), big, None) == 1
    assert lib.sfc_conv2d_nchw(h, C.c_void_p(257), C.c_float(1.0), C.c_void_p(512), C.c_void_p(1024), big, None) == 1
    assert lib.sfc_conv2d_nchw(h, C.c_void_p(256), C.c_float(-1.0), C.c_void_p(512), C.c_void_p(1024), big, None) == 1
    ws = (C.c_float * 24)(*([0.01] * 24))
    assert lib.sfc_transform_filter(h, C.c_void_p(3), ws, C.c_void_p(512), big, None) == 1
    lib.sfc_plan_destroy(h)
    # requantized mode needs its scales before the filter transform
    st, h = plan_status(lib, make_desc())
    assert lib.sfc_transform_filter(h, C.c_void_p(256), ws, C.c_void_p(512), big, None) == 4
    lib.sfc_plan_destroy(h)
    # exact-mode plans take no point scales
    st, h = plan_status(lib, make_desc(mode=0))
    assert lib.sfc_set_point_scales(h, sx, sw) == 2
    lib.sfc_plan_destroy(h)
    assert lib.sfc_status_string(0) == b"ok" and lib.sfc_status_string(4) == b"scales or filter not set"


@pytest.fixture(scope="module")
def kernel_maps(tmp_path_factory):
    """The linear maps realized by the kernels' add networks, compiled for the host."""
    exe = tmp_path_factory.mktemp("host") / "points_check"
    src = os.path.join(ROOT, "tests", "host", "points_check.cpp")
    subprocess.run(["/opt/rocm/bin/hipcc", "--cuda-host-only", "-O1", "-std=c++17", src, "-o", str(exe)],
                   check=True, capture_output=True)
    out = subprocess.run([str(exe)], check=True, capture_output=True, text=True).stdout
    maps = {}
    for line in out.splitlines():
        kind, alg, p, *vals = line.split()
        maps.setdefault((kind, int(alg)), {})[int(p)] = [int(v) for v in vals]
    return {k: np.array([v[i] for i in range(len(v))]) for k, v in maps.items()}


@pytest.mark.parametrize("alg_id,alg", [(0, "6x6_p88"), (1, "6x6_p100"), (2, "7x7_p132"), (3, "7x7_p144"),
                                        (4, "4x4_p46"), (5, "4x4_p49"),
                                        (6, "6x6_5x5_p184"), (7, "6x6_5x5_p196"),
                                        (8, "4x4_7x7_p184"), (9, "4x4_7x7_p196")])
def test_kernel_add_networks_realize_the_oracle_matrices(kernel_maps, alg_id, alg):
    b2, g2, a2, den = oracle.algorithm(alg)
    assert den == (16 if alg in ("4x4_p46", "4x4_p49") else 36)
    assert np.array_equal(kernel_maps[("B", alg_id)], b2)
    assert np.array_equal(kernel_maps[("G", alg_id)], g2)
    assert np.array_equal(kernel_maps[("A", alg_id)], a2)
    # the streaming form of the fused kernels (processing order + per-group collapse)
    assert np.array_equal(kernel_maps[("S", alg_id)], a2)
    if alg_id in (4, 5, 8):  # the form that keeps the outputs instead of the horizontal components
        assert np.array_equal(kernel_maps[("O", alg_id)], a2)


def test_kept_outputs_of_the_5x5_form(kernel_maps):
    """The form with six outputs an axis that keeps the outputs (two pairs per lane)."""
    assert np.array_equal(kernel_maps[("O", 6)], oracle.algorithm("6x6_5x5_p184")[2])


@pytest.mark.parametrize("alg_id", [4, 5])
def test_sfc4_output_transforms_round_alike(kernel_maps, alg_id):
    """Every form of the SFC-4 output transform adds its float32 values in one order: outputs, and
    int8 activations at a tie of their rounding, do not depend on the kernel that a layer runs."""
    assert kernel_maps[("F", alg_id)][0].tolist() == [0, 16000]


@pytest.fixture(scope="module")
def routes(tmp_path_factory):
    """(path, algorithm, shape) of layers -> the product kernels the built library picks for them, or
    (column 1) the output transforms of their exact mode, (2) the forms of single16_kernel, or the input
    kernels, (3) requantized and (4) exact."""
    from paper_2407_02913_amd import binding

    exe = tmp_path_factory.mktemp("host") / "route"
    src = os.path.join(ROOT, "tests", "host", "route.cpp")
    where = os.path.dirname(binding.LIB_PATH)
    subprocess.run(["/opt/rocm/bin/hipcc", "--cuda-host-only", "-O1", "-std=c++17", src, "-L", where,
                    "-l:" + os.path.basename(binding.LIB_PATH), "-Wl,-rpath," + where, "-o", str(exe)],
                   check=True, capture_output=True)

    def ask(layers, column=0):
        text = "".join(f"{binding.PATH[path]} {binding.ALG[alg]} {' '.join(map(str, shape))}\n"
                       for path, alg, shape in layers)
        out = subprocess.run([str(exe)], input=text, check=True, capture_output=True, text=True).stdout
        return [line.split()[column] for line in out.splitlines()]

    return ask


def test_kernels_of_the_shapes_past_the_small_layers(lib, routes):
    """The shapes of the GPU parity test run the kernels they are there for; one image of the same
    geometry runs a kernel for small layers where there is one."""
    import test_gpu_parity as parity

    cases = parity.PAST_SMALL_LAYERS
    assert routes([(path, "4x4_p46", shape) for path, _, shape in cases]) == [kernel for _, kernel, _ in cases]
    one = routes([(path, "4x4_p46", (1, *shape[1:])) for path, _, shape in cases])
    for (path, _, shape), kernel in zip(cases, one):
        small = "single_small" if path == "single" else "product_small" if shape[1] > 128 else "fused_quad"
        assert kernel == small, shape


def test_single16_forms_of_the_parity_shapes(lib, routes):
    """Both forms of single16_kernel, for few workgroups and for many, have shapes of the GPU parity
    tests with one chunk of 64 channels and with two; the lines between them."""
    import test_gpu_parity as parity

    for alg, shapes in (("4x4_p46", [s for _, kernel, s in parity.PAST_SMALL_LAYERS if kernel == "single16"]),
                        ("4x4_p49", parity.SINGLE16_49)):
        forms = routes([("single", alg, s) for s in shapes], column=2)
        seen = {(1 if s[1] <= 64 else 2, form) for s, form in zip(shapes, forms)}
        assert seen == {(1, "few"), (1, "many"), (2, "many")} | ({(2, "few")} if alg == "4x4_p46" else set()), alg
        assert sum(f == "many" for f in forms) >= 5 and len({s[4] % 4 for s, f in zip(shapes, forms) if f == "many"}) >= 3
        # images of 16 tiles: one workgroup each and 64 filters a chunk
        for cin, line in ((64, 512 if alg == "4x4_p46" else 256), (128, 256)):
            layers = [("single", alg, (n, cin, c, 16, 16)) for n, c in
                      ((line, cin), (line // 2, cin + 1), (line + 1, cin), (line // 2 + 1, cin + 1))]
            few = "many" if (alg, cin) == ("4x4_p49", 128) else "few"  # (one form)
            assert routes(layers, column=2) == [few, few, "many", "many"], (alg, cin)


@pytest.mark.parametrize("cin,edge,cout,line", [
    (129, 8, 64, 40), (192, 8, 16, 40), (160, 7, 64, 160), (256, 8, 64, 48), (200, 7, 128, 168), (320, 8, 72, 140),
    (384, 8, 64, 165), (330, 7, 64, 285), (448, 8, 200, 200), (512, 8, 128, 180), (500, 7, 64, 300)])
def test_46_points_quad16_on_both_sides_of_its_line(lib, routes, cin, edge, cout, line):
    """Three to eight chunks of channels: the fused path from a number of workgroups on where its other
    kernels do not take the chunk count, which stays refused on request; quad16_kernel there in any case."""
    from paper_2407_02913_amd import binding

    groups = -(-cout // 64)
    for blocks, here in ((-(-line // groups) - 1, False), (-(-line // groups), True)):
        shape = (4 * blocks, cin, cout, edge, edge)
        assert (routes([("fused", "4x4_p46", shape)]) == ["quad16"]) == here, blocks
        plan = binding.Plan(*shape, alg="4x4_p46", mode="requant", path="auto")
        odd = -(-cin // 64) in (3, 5, 6, 7)
        assert plan.path == ("fused" if here or not odd else "staged"), blocks
        plan.close()
        if odd:
            with pytest.raises(binding.SfcError) as e:
                binding.Plan(*shape, alg="4x4_p46", mode="requant", path="fused")
            assert e.value.code == 2
    few = (4 * 600, cin, 39, edge, edge)  # fewer than 5/8 of a workgroup's filters
    assert (routes([("fused", "4x4_p46", few)]) == ["quad16"]) == (cin <= 320)


def test_kernels_of_the_wide_46_point_shapes(lib, routes):
    import test_gpu_parity as parity

    assert set(routes([("fused", "4x4_p46", shape) for shape in parity.QUAD16_WIDE])) == {"quad16"}


def test_kernels_of_the_184_point_shapes(lib, routes):
    import test_gpu_parity as parity

    cases = parity.SHAPES_184
    assert routes([("fused", "4x4_7x7_p184", shape) for _, shape in cases]) == [kernel for kernel, _ in cases]


def test_kernels_of_the_5x5_shapes(lib, routes):
    import test_gpu_parity as parity

    assert set(routes([("fused", "6x6_5x5_p184", shape) for shape in parity.PAIR16_SHAPES])) == {"pair16"}
    assert set(routes([("fused", "6x6_5x5_p196", shape) for shape in parity.PAIR16_SHAPES])) == {"fused_quad"}


@pytest.mark.parametrize("alg,cin,cout,line", [
    ("6x6_5x5_p184", 64, 64, 36), ("6x6_5x5_p184", 64, 32, 8), ("6x6_5x5_p184", 100, 128, 64),
    ("6x6_5x5_p184", 129, 64, 92), ("6x6_5x5_p184", 257, 300, 130), ("6x6_5x5_p184", 512, 64, 170),
    ("4x4_7x7_p184", 30, 64, 18), ("4x4_7x7_p184", 128, 40, 60), ("4x4_7x7_p184", 150, 64, 80),
    ("4x4_7x7_p184", 256, 128, 100), ("4x4_7x7_p184", 512, 256, 200)])
def test_auto_path_on_both_sides_of_its_line(lib, alg, cin, cout, line):
    """Layers with 184 points: three kernels below a number of workgroups, the fused path from there on;
    the chunk counts that the fused path refuses on request stay refused."""
    from paper_2407_02913_amd import binding

    edge, groups = int(alg[0]), -(-cout // 64)
    for blocks, path in ((-(-line // groups) - 1, "staged"), (-(-line // groups), "fused")):
        plan = binding.Plan(16 * blocks, cin, cout, edge, edge, alg=alg, mode="requant", path="auto")
        assert plan.path == path, blocks
        plan.close()
    if -(-cin // 64) in (1, 2, 4, 8):
        binding.Plan(1, cin, cout, edge, edge, alg=alg, mode="requant", path="fused").close()
    else:
        with pytest.raises(binding.SfcError) as e:
            binding.Plan(1, cin, cout, edge, edge, alg=alg, mode="requant", path="fused")
        assert e.value.code == 2


@pytest.mark.parametrize("cin,cout,tiles", [(64, 64, 64), (30, 40, 64), (64, 128, 32), (60, 300, 1)])
def test_auto_path_of_5x5_filters_with_one_chunk(lib, cin, cout, tiles):
    """Maps of more than one tile: the fused path from five workgroups on, there ahead of three kernels."""
    from paper_2407_02913_amd import binding

    for n, path in ((tiles // 4, "staged"), (tiles // 4 + 1, "fused"), (9 * tiles // 4 + 1, "fused")):
        if n:
            plan = binding.Plan(n, cin, cout, 12, 11, alg="6x6_5x5_p184", mode="requant", path="auto")
            assert plan.path == path, n
            plan.close()


def test_a_stored_choice_gives_the_same_path_again(lib):
    """By its algorithm and SFC_PATH_AUTO, also where the path itself may not be asked for."""
    from paper_2407_02913_amd import binding

    asked = set()
    for alg in ("auto", "4x4_p46", "6x6_5x5_p184", "4x4_7x7_p184", "6x6_p88"):
        for n in (1, 40, 400):
            for cin in (16, 130, 192, 256, 320, 450, 512):
                for edge in (7, 14, 30):
                    plan = binding.Plan(n, cin, 70, edge, edge, alg=alg, mode="requant", path="auto")
                    again = binding.Plan(n, cin, 70, edge, edge, alg=plan.alg, mode="requant", path="auto")
                    assert (again.alg, again.path, again.workspace_bytes) == (plan.alg, plan.path, plan.workspace_bytes)
                    try:
                        binding.Plan(n, cin, 70, edge, edge, alg=plan.alg, mode="requant", path=plan.path).close()
                        asked.add(True)
                    except binding.SfcError as e:
                        assert e.code == 2 and plan.path == "fused" and -(-cin // 64) in (3, 5, 6, 7)
                        asked.add(False)
                    plan.close()
                    again.close()
    assert asked == {True, False}


def test_waves_of_the_5x5_kernel(lib):
    """Four up to 128 workgroups of 64 filters, then eight: the operand covers whole workgroups."""
    from paper_2407_02913_amd import binding
    import test_gpu_parity as parity

    def filters(shape):
        plan = binding.Plan(*shape, alg="6x6_5x5_p184", mode="requant", path="fused")
        cp, kp = -(-shape[1] // 64) * 64, -(-shape[2] // 16) * 16
        # U, the operand, the factors of points (twice) and of positions, the other tables
        rest = plan.filter_bytes - 184 * kp * (cp + 8)
        plan.close()
        return rest // (184 * (cp + 4)) // 16 * 16

    for cin in (64, 512):
        assert filters((16 * 64, cin, 65, 6, 6)) == 96 and filters((16 * 64 + 1, cin, 65, 6, 6)) == 128
    assert {-(-s[2] // 64) * 64 == filters(s) for s in parity.PAIR16_EIGHT_WAVES} == {True}


def test_static_workspace_of_layers_sent_through_m(lib, routes):
    """A layer that the library sends through M and whose V and M exceed the static workspace: at most three passes, and
    those with eight chunks of channels; else its plan holds the fused kernel's operand as well."""
    from paper_2407_02913_amd import binding
    import test_gpu_parity as parity

    assert routes([("fused", alg, s) for alg, s, _, _ in parity.SENT_THROUGH_M]) == [k for _, _, k, _ in parity.SENT_THROUGH_M]
    more = [("4x4_7x7_p184", (20, 512, 576, 16, 16), None, "fused"), ("6x6_5x5_p184", (16, 512, 256, 24, 24), None, "fused"),
            ("6x6_5x5_p184", (16, 512, 192, 24, 24), None, "passes"), ("6x6_5x5_p184", (30, 128, 128, 24, 24), None, "fused"),
            ("6x6_5x5_p184", (4, 512, 64, 12, 12), None, "whole"), ("4x4_7x7_p184", (23, 512, 64, 16, 16), None, "refused")]
    for alg, shape, _, static in parity.SENT_THROUGH_M + more:
        plan = binding.Plan(*shape, alg=alg, mode="requant", path="auto")
        cp, kp = -(-shape[1] // 64) * 64, -(-shape[2] // 16) * 16
        operand = 184 * kp * cp
        assert plan.path == "staged"
        assert (plan.workspace_bytes > binding.STATIC_WORKSPACE_BYTES) == (static != "whole"), shape
        assert (plan.filter_bytes > 2 * operand) == (static == "fused"), shape
        plan.close()


def test_output_transforms_of_the_exact_shapes(lib, routes):
    """Either output transform has the shapes of the GPU parity tests that are there for it."""
    import test_gpu_parity as parity

    cases = parity.EXACT_WAVE_SHAPES
    assert set(routes([("staged", alg, shape) for alg, shape in cases], column=1)) == {"waves"}
    small = [("staged", alg, shape) for alg in parity.ALGS_STAGED + parity.ALGS_5X5 for shape in parity.SMALL_SHAPES
             if shape != (5, 64, 64, 12, 18)]
    assert set(routes(small, column=1)) == {"threads"}
    # the lines: 9 to 15 filters, 16 to 63, 64 and more with even and with odd width
    for alg, *lines in (("6x6_p88", 2560, 1025, 768, 1200), ("7x7_p132", 2560, 768, 0, 48),
                        ("4x4_p46", 4096, 1024, 512, 768), ("6x6_5x5_p184", None, 2560, 48, 640),
                        ("4x4_7x7_p184", None, 4096, 160, 640)):
        for cout, width, line in zip((9, 16, 63, 64, 300), (4, 4, 3, 4, 3), (*lines[:2], *lines[1:])):
            if line is None:
                assert routes([("staged", alg, (200000, 1, 15, 4, 4))], column=1) == ["threads"]
                continue
            images = max(1, -(-16 * line // -(-cout // 4)))  # one tile each
            layers = [("staged", alg, (images - i, 1, cout, 4, width)) for i in (0, 1) if images > i]
            assert routes(layers, column=1) == ["waves", "threads"][: len(layers)], (alg, cout)
        assert routes([("staged", alg, (200000, 1, 8, 4, 4))], column=1) == ["threads"]


def test_row_form_takes_every_algorithm(lib, routes):
    """The row-form input transform, whose GPU test compares V: exact mode on any map, requantized mode
    outside small ones."""
    import test_gpu_parity as parity

    algs = parity.ALGS_STAGED + parity.ALGS_5X5
    large = parity.ROWS_SHAPES[1:] + [(2, 64, 3, 224, 224), (1, 512, 3, 40, 1024)]
    small = parity.ROWS_SHAPES[:1] + [(256, 64, 3, 7, 7), (1, 1, 1, 1, 1), (64, 256, 3, 14, 14)]
    assert set(routes([("staged", alg, shape) for alg in algs for shape in large + small], column=4)) == {"rows"}
    assert set(routes([("staged", alg, shape) for alg in algs for shape in large], column=3)) == {"rows"}
    assert routes([("staged", alg, (64, 256, 3, 14, 14)) for alg in ("6x6_p88", "4x4_p46", "4x4_7x7_p184")],
                  column=3) == ["image", "waves", "rows"]


def test_every_kernel_choice_fits_the_filter_layout(lib, routes):
    """Single path: the kernel for small layers reads the operand of the 16-filter kernels, and is
    only picked where one of those would be without it."""
    shapes = [(n, cin, cout, h, w) for n in (1, 3, 40) for cin in (1, 16, 64, 65, 128) for cout in (1, 40, 300)
              for h, w in ((1, 1), (7, 7), (13, 9), (56, 56), (9, 200), (300, 5), (4, 1024))]
    for shape, kernel, kernel49 in zip(shapes, routes([("single", "4x4_p46", s) for s in shapes]),
                                       routes([("single", "4x4_p49", s) for s in shapes])):
        assert kernel in ("single_small", "single16"), (shape, kernel)
        assert kernel49 == "single16", (shape, kernel49)


def kernel_resources(path):
    """(kernel, scratch bytes of a lane, spilled vector registers) of every gfx950 kernel in a library,
    from the metadata notes of its code objects."""
    readelf = "/opt/rocm/llvm/bin/llvm-readelf"
    data = open(path, "rb").read()
    magic = b"__CLANG_OFFLOAD_BUNDLE__"
    start, found = data.find(magic), []
    while start >= 0:
        count, = struct.unpack_from("<Q", data, start + len(magic))
        at = start + len(magic) + 8
        for _ in range(count):
            offset, size, name = struct.unpack_from("<QQQ", data, at)
            target = data[at + 24 : at + 24 + name].decode()
            at += 24 + name
            if size and "gfx950" in target:
                notes = subprocess.run([readelf, "--notes", "-"], input=data[start + offset : start + offset + size],
                                       check=True, capture_output=True).stdout.decode()
                # (a kernel's keys are sorted, .name before .private_segment_fixed_size)
                found += re.findall(r"\n    \.name: +(\S+)\n.*?\.private_segment_fixed_size: (\d+)\n.*?"
                                    r"\.vgpr_spill_count: (\d+)", notes, flags=re.S)
        start = data.find(magic, at)
    names = subprocess.run(["c++filt"], input="\n".join(k for k, _, _ in found), check=True, capture_output=True,
                           text=True).stdout.splitlines()
    return [(name, int(scratch), int(spilled)) for name, (_, scratch, spilled) in zip(names, found)]


def test_single16_keeps_its_values_in_registers(lib):
    """No form of single16_kernel works in scratch memory; the one for 46 points, two chunks and many
    workgroups keeps a few values there, each written and read once (Single16Ahead)."""
    from paper_2407_02913_amd import binding

    kernels = {name[: name.index("(")]: rest for name, *rest in kernel_resources(binding.LIB_PATH)
               if "single16_kernel<" in name}
    assert {name.split("<")[1][:4] for name in kernels} == {"4, 1", "4, 2", "5, 1", "5, 2"}
    for name, (scratch, spilled) in kernels.items():
        few = "single16_kernel<4, 2," in name and name.endswith("false>")
        assert scratch <= (48 if few else 0) and spilled <= (12 if few else 0), (name, scratch, spilled)


def test_bench_operation_counts_match_the_add_networks(tmp_path):
    """bench.py's vector-ALU roofline counts: recounted from sfc_points.hpp with a counting type."""
    import bench

    exe = tmp_path / "op_count"
    src = os.path.join(ROOT, "tests", "host", "op_count.cpp")
    subprocess.run(["/opt/rocm/bin/hipcc", "--cuda-host-only", "-O1", "-std=c++17", src, "-o", str(exe)],
                   check=True, capture_output=True)
    out = subprocess.run([str(exe)], check=True, capture_output=True, text=True).stdout
    names = ["6x6_p88", "6x6_p100", "7x7_p132", "7x7_p144", "4x4_p46", "4x4_p49"]
    for line in out.splitlines():
        alg, pts, in_adds, out_ops = (int(v) for v in line.split())
        assert pts == oracle.multiplications_per_tile(names[alg])
        assert bench.ADD_NETWORK_OPS[names[alg]] == (in_adds, out_ops)
    # the 6x6 input network is the paper's: 14 additions per symbolic DFT-6 plus the correction
    # inputs, 16 per 1-D pass over 8 + 8 lines, plus the sums of the product rule
    assert bench.ADD_NETWORK_OPS["6x6_p88"][0] == 16 * 16 + 48


def test_group_scales_matches_the_oracle_for_every_granularity(lib):
    """Host-only entry point: the ablation's scale groupings against the oracle's."""
    from paper_2407_02913_amd import binding

    rng = np.random.default_rng(5)
    plan = binding.Plan(2, 16, 24, 14, 9, alg="6x6_p88", mode="requant")
    sx = rng.uniform(0.1, 4.0, size=plan.P).astype(np.float32)
    sw = rng.uniform(0.1, 4.0, size=(plan.P, 24)).astype(np.float32)
    for act in ("tensor", "point"):
        for filt in ("channel", "point", "channel_point"):
            gx, gw = plan.group_scales(sx, sw, act, filt)
            ox, ow = oracle.group_scales(sx, sw, act, filt)
            assert np.array_equal(gx, ox) and np.array_equal(gw, ow), (act, filt)
    h = plan._h
    fx, fw = (C.c_float * plan.P)(), (C.c_float * (plan.P * 24))()
    assert lib.sfc_group_scales(h, 2, 0, fx, fw) == 1 and lib.sfc_group_scales(h, 0, 3, fx, fw) == 1
    assert lib.sfc_group_scales(h, 0, 0, None, fw) == 1
    plan.close()
