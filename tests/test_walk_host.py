"""What the host says about how a call is walked (sr_dict_assemble_walk, sr_dict_assemble_list_walk): tiles or strips, as
launched.  No GPU and no launch: descriptors with fake, well-separated device addresses."""
import ctypes

import pytest

import paper_2303_08999_amd as sr

DT = {"f16": sr.SR_F16, "bf16": sr.SR_BF16, "f8": sr.SR_F8E4M3, "f32": sr.SR_F32}
TILES, STRIPS = 1, 2


def _far(*tensors):
    return [sr.sr_tensor(0x1000000000 * (i + 1), *t) for i, t in enumerate(tensors)]


def walk(n=1, C=3, H=2160, W=3840, s=4, L=72, k=5, cd="f16", kept=None, opts=None, kind=sr.SR_COEFF_VALUES, kernel=sr.SR_KERNEL_AUTO, tile=0):
    lr, coeff, d, out = _far((sr.SR_F32, n, C, H // s, W // s), (DT[cd], n, L, H, W), (sr.SR_F32, 1, L, k, k), (sr.SR_F32, n, C, H, W))
    ka = (ctypes.c_int * len(kept))(*kept) if kept else None
    w = (ctypes.c_int * 6)(*[-1] * 6)
    st = sr.load().sr_dict_assemble_walk(lr, coeff, d, L, k, s, C, out, ka, len(kept or ()),
                                         ctypes.byref(opts or sr.make_options(kernel, tile, coeff_kind=kind)), w)
    return st, tuple(w)


def list_walk(n=1, H=2160, W=3840, s=4, L=72, entries=8, value="f16", kernel=sr.SR_KERNEL_AUTO):
    ts = _far((sr.SR_F32, n, 3, H // s, W // s), (sr.SR_U8, n, entries, H, W), (DT[value], n, entries, H, W), (sr.SR_F32, 1, L, 5, 5),
              (sr.SR_F32, n, 3, H, W))
    w = (ctypes.c_int * 6)(*[-1] * 6)
    st = sr.load().sr_dict_assemble_list_walk(*ts[:4], L, 5, s, 3, entries, ts[4], kernel, w)
    return st, tuple(w)


def _whole(w, n, H, W):
    """The pieces cover the images, and the launch has work for all of its workgroups."""
    form, width, rows, pieces, workgroups, waves = w
    assert pieces == n * -(-W // width) * -(-H // rows)
    assert workgroups * (waves if form == STRIPS else 1) < pieces + waves


@pytest.mark.parametrize("cd", list(DT))
@pytest.mark.parametrize("k, C, L", [(3, 1, 72), (3, 3, 128), (5, 1, 72), (5, 3, 8), (5, 3, 40), (5, 3, 72), (5, 3, 128), (7, 1, 72), (7, 3, 128)])
@pytest.mark.parametrize("s", [2, 3, 4])
def test_every_call_of_the_matrix_core_kernel_has_a_walk(cd, k, C, L, s):
    forms = set()
    for n, h, w in ((1, 8, 32), (1, 128, 128), (3, 77, 60), (1, 360, 640), (16, 270, 480), (1, 360, 641)):
        H, W = h * s, w * s
        kernel, got = walk(n=n, C=C, H=H, W=W, s=s, L=L, k=k, cd=cd)
        if kernel == sr.SR_KERNEL_GENERIC:
            assert got == (0,) * 6
            continue
        assert kernel == sr.SR_KERNEL_MFMA and got[0] in (TILES, STRIPS)
        _whole(got, n, H, W)
        forms.add(got[0])
    assert forms or (k == 7 and L <= 16) or cd in ("f8", "f32")


def test_a_tile_index_is_walked_in_its_tiles():
    """Index 0 may be strips; every other index is the tile that sr_dict_assemble_launch_shape reports for it."""
    for tile in range(1, 10):
        lr, coeff, d, out = _far((sr.SR_F32, 1, 3, 540, 960), (sr.SR_F16, 1, 72, 2160, 3840), (sr.SR_F32, 1, 72, 5, 5),
                                 (sr.SR_F32, 1, 3, 2160, 3840))
        shape = (ctypes.c_int * 4)()
        opts = sr.make_options(sr.SR_KERNEL_MFMA, tile)
        assert sr.load().sr_dict_assemble_launch_shape(lr, coeff, d, 72, 5, 4, 3, out, None, 0, ctypes.byref(opts), shape) == sr.SR_KERNEL_MFMA
        kernel, got = walk(opts=opts)
        assert kernel == sr.SR_KERNEL_MFMA and got[:3] == (TILES, shape[0], shape[1]) and got[5] == shape[2]
        _whole(got, 1, 2160, 3840)
    assert walk()[1][:3] == (STRIPS, 128, 32)            # the 4K frame's default


def test_walk_statuses():
    assert walk(kernel=sr.SR_KERNEL_GENERIC) == (sr.SR_KERNEL_GENERIC, (0,) * 6)
    assert walk(C=2, cd="f32") == (sr.SR_KERNEL_GENERIC, (0,) * 6)
    assert walk(H=0) == (sr.SR_KERNEL_GENERIC, (0,) * 6)
    assert walk(tile=10)[0] == walk(C=2, cd="f32", kernel=sr.SR_KERNEL_MFMA)[0] == -3
    assert walk(kept=[72])[0] < 0
    assert list_walk(kernel=sr.SR_KERNEL_GENERIC) == (sr.SR_KERNEL_GENERIC, (0,) * 6)
    assert list_walk(value="f32") == (sr.SR_KERNEL_GENERIC, (0,) * 6)
    assert list_walk(value="f32", kernel=sr.SR_KERNEL_MFMA)[0] == list_walk(kernel=3)[0] == -3
    for s in (2, 3, 4):
        for L in (72, 128):
            for n, h, w in ((1, 8, 32), (1, 180, 320), (4, 270, 480)):
                kernel, got = list_walk(n=n, H=h * s, W=w * s, s=s, L=L)
                assert kernel == sr.SR_KERNEL_MFMA and got[0] in (TILES, STRIPS)
                _whole(got, n, h * s, w * s)
    lr, coeff, d, out = _far((sr.SR_F32, 1, 3, 8, 32), (sr.SR_F16, 1, 72, 32, 128), (sr.SR_F32, 1, 72, 5, 5), (sr.SR_F32, 1, 3, 32, 128))
    assert sr.load().sr_dict_assemble_walk(lr, coeff, d, 72, 5, 4, 3, out, None, 0, None, None) == -1


@pytest.mark.parametrize("H, W, s", [(720, 960, 4), (768, 1024, 4), (800, 800, 4), (540, 960, 4), (512, 1280, 4)])
def test_8_bit_frames_that_strips_refuse_take_the_tile_they_were_compared_with(H, W, s):
    """72 atoms, three channels, x4, about 0.4 to 0.8 Mpixel: strips and 128 x 24 tiles leave the fullest SIMD six rows;
    128 x 16 tiles would leave it eight."""
    kernel, got = walk(H=H, W=W, s=s, cd="f8")
    assert kernel == sr.SR_KERNEL_MFMA and (got[0] == STRIPS or got[:3] == (TILES, 128, 24))


@pytest.mark.parametrize("n, H, W", [(1, 4, 4), (1, 480, 640), (1, 720, 1280), (1, 800, 1200), (32, 128, 192), (1, 2160, 3840), (4000, 8, 16)])
@pytest.mark.parametrize("entries", [8, 16])
def test_lists_of_up_to_72_atoms_at_scale_4_take_strips(n, H, W, entries):
    kernel, got = list_walk(n=n, H=H, W=W, entries=entries)
    assert kernel == sr.SR_KERNEL_MFMA and got[:2] == (STRIPS, 128)
    _whole(got, n, H, W)


@pytest.mark.parametrize("call, form", [
    # rows of whole 128-byte lines: strips at about the same number of rows of the fullest SIMD
    (dict(), STRIPS), (dict(H=1536, W=2048, s=2), STRIPS), (dict(H=1536, W=2048, L=128, k=7), STRIPS), (dict(cd="f8"), STRIPS),
    # rows that share lines, the stream as the bound: tiles unless strips save 8 %
    (dict(W=3816), TILES), (dict(W=3816, cd="f8"), TILES), (dict(W=3816, cd="bf16", kind=sr.SR_COEFF_LOGITS), TILES),
    (dict(H=1536, W=2040, s=2), TILES), (dict(H=1536, W=2040, s=3, k=7, C=1), TILES), (dict(H=1536, W=2040, s=3, cd="f32", C=1), TILES),
    (dict(H=1200, W=1600, s=2, L=128), STRIPS), (dict(H=1200, W=1608, s=2, L=128), TILES), (dict(H=1536, W=2040, C=1, kept=list(range(30))), TILES),
    # ... not bound by it: half lines, fewer coefficients than the memory-side cache holds, wavefronts to spare, capacity to spare, fp32 with 7x7 atoms
    (dict(H=1800, W=3232, L=128), STRIPS), (dict(H=540, W=936, s=2), STRIPS), (dict(H=900, W=1600, s=2, cd="f8", kept=list(range(45))), STRIPS),
    (dict(H=1200, W=1608), STRIPS), (dict(H=1536, W=2040, s=2, L=52), STRIPS), (dict(H=1200, W=1596, s=3, k=7, cd="f32"), STRIPS),
    # ... few atoms, or three channels and 30 atoms: the up-sampling counts, strips as before
    (dict(W=3816, kept=list(range(8))), STRIPS), (dict(H=1536, W=2040, kept=list(range(30))), STRIPS),
    # scale 3, segments of one row against tiles of two
    (dict(H=240, W=312, s=3, kept=[0, 9]), TILES), (dict(H=144, W=192, s=3, cd="f8", L=8), TILES),
    (dict(H=444, W=714, s=3, C=1, cd="f32", L=8), TILES), (dict(H=444, W=714, s=3, cd="f32", L=8), STRIPS), (dict(H=480, W=636, s=3, C=1, k=7), STRIPS),
    (dict(H=240, W=312, s=2, kept=[0, 9]), STRIPS), (dict(H=240, W=312, s=3, L=40), STRIPS),
])
def test_which_form_a_call_takes(call, form):
    assert walk(**call)[1][0] == form


@pytest.mark.parametrize("cd", list(DT))
@pytest.mark.parametrize("kind", [sr.SR_COEFF_VALUES, sr.SR_COEFF_LOGITS])
def test_no_strip_starts_between_its_first_columns(cd, kind):
    """A last strip that is moved left to end at the image edge starts at column 0 or at R or beyond: the strip form continues
    the image on the left of column 0 for a strip that starts there only."""
    for k, C, L in ((3, 1, 72), (3, 3, 8), (5, 1, 72), (5, 3, 8), (5, 3, 30), (5, 3, 72), (5, 3, 128), (7, 1, 72), (7, 3, 12)):
        for n, h in ((1, 1), (1, 43), (32, 43), (400, 43), (1, 3000)):
            for w in range(43, 68):
                form, width = walk(n=n, C=C, H=3 * h, W=3 * w, s=3, L=L, k=k, cd=cd, kind=kind)[1][:2]
                if form == STRIPS and (3 * w) % (width // 32) != 0:
                    assert 3 * w - width == 0 or 3 * w - width >= k // 2, (k, C, L, n, h, w)


def test_images_up_to_4_gb_are_the_matrix_core_kernels():
    """The last 64 bytes below 4 GB included; an odd number of 2^30 - 1 pixels in strips, whose lanes are all inside the image."""
    H, W = 2 * 16383, 2 * 16385
    assert H * W == (1 << 30) - 4
    for kernel in (sr.SR_KERNEL_AUTO, sr.SR_KERNEL_MFMA):
        for cd, L in (("f8", 3), ("f16", 1), ("bf16", 1)):
            assert walk(C=1, H=H, W=W, s=2, L=L, cd=cd, kernel=kernel)[0] == sr.SR_KERNEL_MFMA
    H, W = 3 * 7 * 11 * 331, 3 * 31 * 151
    assert H * W == (1 << 30) - 1
    for k in (3, 5):
        for cd, L in (("f8", 4), ("f16", 2), ("bf16", 2)):
            assert walk(C=1, H=H, W=W, s=3, L=L, k=k, cd=cd, kernel=sr.SR_KERNEL_MFMA)[1][0] == STRIPS
    assert walk(C=1, H=1 << 15, W=1 << 15, s=2, L=1, cd="f8", kernel=sr.SR_KERNEL_MFMA)[0] == -3


def _apart(*tensors):
    """_far for tensors of many terabytes."""
    return [sr.sr_tensor((i + 1) << 52, *t) for i, t in enumerate(tensors)]


def runs(n=1, C=3, H=2160, W=3840, s=4, L=72, k=5, cd="f16", kept=None, pre=False, logits=False, kernel=sr.SR_KERNEL_AUTO, tile=0):
    lr, coeff, d, out = _apart((sr.SR_F32, n, C, H // s, W // s), (DT[cd], n, L * s * s, H // s, W // s) if pre else (DT[cd], n, L, H, W),
                             (sr.SR_F32, 1, L, k, k), (sr.SR_F32, n, C, H, W))
    opts = sr.make_options(kernel, tile, sr.SR_COEFF_PRE_SHUFFLE if pre else sr.SR_COEFF_PLANAR, sr.SR_COEFF_LOGITS if logits else sr.SR_COEFF_VALUES)
    ka = (ctypes.c_int * len(kept))(*kept) if kept else None
    w = (ctypes.c_int * 6)(*[-1] * 6)
    return sr.load().sr_dict_assemble_runs(lr, coeff, d, L, k, s, C, out, ka, len(kept or ()), ctypes.byref(opts), w), tuple(w)


def test_the_kernel_that_is_launched():
    """Where sr_dict_assemble_plan knows two answers, sr_dict_assemble_runs knows three, and the walk of both matrix-core kernels."""
    assert runs() == (sr.SR_RUNS_STREAMING, walk()[1])
    assert runs(kernel=sr.SR_KERNEL_GENERIC) == (sr.SR_RUNS_GENERIC, (0,) * 6)
    assert runs(H=0) == (sr.SR_RUNS_NOTHING, (0,) * 6)
    assert runs(tile=10)[0] == runs(C=2, cd="f32", kernel=sr.SR_KERNEL_MFMA)[0] == -3 and runs(kept=[72])[0] < 0
    for call in (dict(C=2, cd="f32"), dict(pre=True, cd="f8"), dict(logits=True, k=3), dict(logits=True, cd="f32", pre=True)):
        kernel, got = runs(**call)
        assert kernel == sr.SR_RUNS_SLOTS and got[0] == TILES
        assert runs(**call, kernel=sr.SR_KERNEL_GENERIC) == (sr.SR_RUNS_GENERIC, (0,) * 6)
    small = dict(C=1, H=128, W=128, s=2, cd="f32")       # a planar call that it has from the streaming kernel
    assert runs(**small) == runs(**small, kernel=sr.SR_KERNEL_MFMA) == (sr.SR_RUNS_SLOTS, walk(**small)[1])
    assert runs(C=5, cd="f16") == runs(L=200) == (sr.SR_RUNS_GENERIC, (0,) * 6)
    lr, coeff, d, out = _far(*[(sr.SR_F32, 1, 3, 8, 8)] * 4)
    assert sr.load().sr_dict_assemble_runs(lr, coeff, d, 72, 5, 4, 3, out, None, 0, None, None) == -1


# calls that the generic kernel serves faster, and the same on the other side of the line
@pytest.mark.parametrize("call, atoms", [
    (dict(C=1, H=600, W=600, s=2, k=5, logits=True), (8, 9)), (dict(C=1, H=600, W=600, s=3, k=7, cd="f32", logits=True, pre=True), (8, 9)),
    (dict(C=2, H=600, W=600, s=4, k=7, cd="bf16", logits=True), (14, 15)), (dict(C=2, H=600, W=600, s=2, k=5, pre=True), (16, 17)),
    (dict(C=1, H=600, W=600, s=2, k=3, cd="bf16", pre=True), (12, 13)), (dict(C=3, H=600, W=600, s=2, k=3, cd="f32", pre=True), (22, 23)),
    (dict(C=3, H=600, W=600, s=2, k=3, cd="f32", pre=True), (33, 32)), (dict(C=3, H=600, W=600, s=2, k=3, cd="f32", pre=True), (42, 43)),
    (dict(C=2, H=600, W=600, s=2, k=5, cd="f32"), (42, 43)), (dict(C=2, H=600, W=600, s=2, k=5, cd="f32"), (20, 21)), (dict(C=2, H=600, W=600, s=2, k=7, cd="f32"), (48, 49)),
    (dict(C=3, H=600, W=600, s=2, k=7, cd="bf16", pre=True), (36, 37)), (dict(C=3, H=600, W=600, s=2, k=7, cd="f8", pre=True), (100, 101))])
def test_calls_that_the_generic_kernel_serves_faster(call, atoms):
    assert runs(L=atoms[0], **call) == (sr.SR_RUNS_GENERIC, (0,) * 6)
    assert runs(L=atoms[1], **call)[0] == sr.SR_RUNS_SLOTS
    if call.get("cd") in ("f32", "f8") and atoms[0] > 25:     # (a small frame: not)
        assert runs(L=atoms[0], **dict(call, H=48, W=72))[0] == sr.SR_RUNS_SLOTS


def test_more_tiles_than_32_bits_count():
    """Thin images in their largest number: the generic kernel, as before, and no refusal."""
    for call in (dict(pre=True, cd="f8"), dict(logits=True, C=1), dict(C=2, cd="f32")):
        assert runs(n=65535, H=262140, W=8, s=2, L=72, **call) == (sr.SR_RUNS_GENERIC, (0,) * 6)
        assert runs(n=600, H=262140, W=8, s=2, L=72, **call)[0] == sr.SR_RUNS_SLOTS


def test_lr_widths_off_multiples_of_4_before_the_pixel_shuffle():
    """fp16, 65 to 72 atoms, HR widths of whole groups: the second matrix-core kernel; a single LR column, whose rows hold no word of coefficients, stays on the streaming
    one's element-wise form, and frames beyond the tile count at scale 2 (more coefficients than a device holds) are the generic kernel's."""
    for s, W in ((4, 8), (4, 20), (4, 132), (2, 4), (2, 12), (2, 1004)):
        for kernel in (sr.SR_KERNEL_AUTO, sr.SR_KERNEL_MFMA):
            assert runs(H=24, W=W, s=s, cd="f16", pre=True, kernel=kernel)[0] == sr.SR_RUNS_SLOTS
    for kernel in (sr.SR_KERNEL_AUTO, sr.SR_KERNEL_MFMA):
        assert runs(H=24, W=4, s=4, cd="f16", pre=True, kernel=kernel) == (sr.SR_RUNS_STREAMING, (TILES, 128, 12, 2, 2, 2))
    beyond = dict(n=65535, H=32800, W=4, s=2, cd="f16", pre=True)
    assert runs(**beyond) == (sr.SR_RUNS_GENERIC, (0,) * 6) and runs(**beyond, kernel=sr.SR_KERNEL_MFMA)[0] == -3
