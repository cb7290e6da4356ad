"""The strip form of the matrix-core kernel where it can go wrong: strips that stick out of the image or end it on an odd
column, every scale (three ways of grouping the columns), first and last rows, rings that turn, several segments per wavefront,
every pixel group and coefficient type; and tiles of about the same sizes.  Which form a call takes depends on the rows
of the fullest SIMD: the first tests take either (frames of about the sizes that change over), those named as_launched
ask sr_dict_assemble_walk first.  Against the generic kernel, whose up-sampled values are the same bit for bit, so that only the
order of fp32 sums and the 16-bit dictionary operands differ: 5e-5 * max(1, max|out|) and 2^-10 of it for an fp16 image,
bfloat16 coefficients 1e-4 (dictionary of 16 significant bits); and the pixels at the borders against the oracle."""
import numpy as np
import pytest
import torch

import paper_2303_08999_amd as sr
import sr_synth
from test_gpu_parity import DEV, GENERIC, MFMA, assert_parity, check_full, run_gpu

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    assert torch.cuda.is_available(), "these tests need the MI355X"
    sr.load()


def _assert_strips(walk, rows, segments):
    """Strips, of segments of at least so many rows, and at least so many of them to a wavefront."""
    kernel, (form, _, got, pieces, workgroups, waves) = walk
    assert kernel == MFMA and form == 2 and got >= rows and pieces > (segments - 1) * workgroups * waves, walk


def _check(oracle, n, c, h, w, scale, L, k, coeff, image, kept, strip_rows=0, segments=0):
    wl = sr_synth.Workload("strips", 60, n, c, h, w, scale, L, k, coeff, image)
    inp = sr_synth.make_inputs(wl, DEV)
    rng = np.random.default_rng(h)
    lst = None if kept is None else rng.permutation(L)[:kept].astype(np.int32)
    gamma = None if kept is None else rng.uniform(0.5, 1.5, size=kept).astype(np.float32)
    if strip_rows:
        out = torch.empty((n, c, wl.H, wl.W), device=DEV, dtype=inp["lr"].dtype)
        _assert_strips(sr.sr_dict_assemble_walk(inp["lr"], inp["coeff"], inp["dict"], L, k, scale, c, out, kept=lst), strip_rows, segments)
    got = run_gpu(inp, wl, MFMA, lst, gamma).float()
    want = run_gpu(inp, wl, GENERIC, lst, gamma).float()
    assert torch.isfinite(got).all(), "some output pixel was never written"
    tol = ((1e-4 if coeff == "bf16" else 5e-5) + (2.0 ** -10 if image == "f16" else 0.0)) * max(1.0, float(want.abs().max()))
    assert float((got - want).abs().max()) <= tol
    if n == 1:
        rows = sorted({0, 1, 2, wl.H // 2, wl.H - 3, wl.H - 2, wl.H - 1})
        pts = np.array([(0, y, x) for y in rows for x in (0, 1, 2, 127, min(128, wl.W - 1), wl.W - 3, wl.W - 2, wl.W - 1)])
        ref = oracle.assemble_points(oracle.bicubic(inp["lr"].cpu().numpy(), scale), sr_synth.stored_numpy(inp["coeff"]),
                                     inp["dict"].cpu().numpy(), pts, kept=lst, gamma=gamma)
        have = got[0].cpu().numpy()[:, pts[:, 1], pts[:, 2]].T
        assert_parity(have, ref, coeff, image == "f16", "borders")


@pytest.mark.parametrize("n, c, h, w, scale, L, k, coeff, image, kept", [
    (1, 3, 270, 480, 4, 72, 5, "f16", "f32", None),      # whole strips
    (1, 3, 271, 473, 4, 72, 5, "f16", "f16", None),      # the last strip sticks out of the image
    (1, 3, 300, 333, 3, 72, 5, "f8", "f32", None),       # rows that are no whole pixel groups: the last tile or strip is moved left
    (1, 3, 301, 501, 2, 72, 5, "f16", "f32", None),
    (1, 3, 400, 43, 3, 72, 5, "f16", "f32", None),       # 129 columns: two pieces, almost the same
    (2, 3, 301, 501, 2, 72, 5, "f32", "f16", None),
    (1, 1, 501, 301, 3, 72, 5, "f32", "f32", None),
    (3, 3, 190, 250, 4, 72, 5, "f16", "f32", 8),         # kept lists: the forms with few planes
    (1, 3, 333, 502, 3, 72, 5, "f8", "f32", 8),
    (1, 3, 301, 502, 2, 72, 5, "bf16", "f32", 13),
    (1, 1, 333, 401, 3, 72, 5, "bf16", "f32", None),
    (1, 3, 250, 330, 4, 128, 5, "f16", "f32", None),     # two pixels per lane
    (1, 3, 250, 331, 3, 128, 7, "f16", "f16", None),     # two matrix blocks per slot
    (1, 1, 251, 401, 2, 72, 7, "bf16", "f32", None),
    (1, 3, 251, 401, 2, 72, 7, "f32", "f32", None),
    (1, 3, 333, 401, 3, 40, 3, "f32", "f32", None),
    (1, 3, 333, 500, 2, 72, 3, "f8", "f16", None),
    (1, 3, 251, 401, 4, 128, 3, "f16", "f32", 30),
    (2300, 3, 4, 16, 2, 72, 5, "f16", "f32", None),      # more strips than wavefronts: several segments one after the other
])
def test_strips(oracle, n, c, h, w, scale, L, k, coeff, image, kept):
    _check(oracle, n, c, h, w, scale, L, k, coeff, image, kept)


# (strip_rows: more than the ring has slots, four, six or eight, so that it turns)
@pytest.mark.parametrize("n, c, h, w, scale, L, k, coeff, image, kept, strip_rows, segments", [
    (1, 3, 419, 257, 3, 128, 7, "f16", "f16", None, 9, 1),     # eight ring rows, groups before the image's first column; the last strip moved left
    (1, 3, 292, 387, 3, 72, 7, "f32", "f32", None, 9, 1),
    (1, 1, 540, 640, 2, 72, 7, "bf16", "f32", None, 9, 1),
    (1, 3, 540, 641, 2, 72, 7, "f32", "f32", None, 9, 1),
    (1, 3, 374, 161, 4, 72, 7, "f16", "f32", 12, 9, 1),
    (1, 3, 305, 171, 3, 40, 3, "f32", "f32", None, 5, 1),      # four ring rows
    (1, 3, 400, 640, 3, 72, 3, "f16", "f16", None, 5, 1),
    (1, 3, 420, 403, 3, 72, 5, "f8", "f32", None, 7, 1),       # six; the last strip moved left
    (1, 3, 413, 398, 3, 72, 5, "f16", "f32", None, 7, 1),
    (1, 1, 375, 215, 3, 72, 5, "f32", "f16", None, 7, 1),
    (1, 3, 1000, 513, 3, 72, 5, "f8", "f32", 8, 7, 1),
    (1, 3, 540, 961, 2, 72, 5, "bf16", "f32", 13, 7, 1),
    (1, 1, 400, 640, 3, 72, 5, "bf16", "f32", None, 7, 1),
    (2435, 3, 2, 4, 3, 72, 5, "f16", "f32", None, 6, 2),       # several segments one after the other: every wavefront of the launch walks one, some two
    (2213, 3, 2, 4, 3, 72, 5, "f32", "f32", None, 6, 2),
    (2125, 3, 2, 5, 2, 72, 7, "f16", "f16", None, 4, 2),
    (4200, 1, 2, 5, 2, 72, 5, "f32", "f32", None, 4, 3),
    (3135, 3, 2, 3, 4, 72, 5, "f16", "f32", 8, 8, 2),          # few planes: their offsets in registers, three wavefronts per SIMD
    (1030, 3, 2, 33, 4, 72, 5, "f8", "f32", None, 8, 2),       # two strips to an image
])
def test_strips_as_launched(oracle, n, c, h, w, scale, L, k, coeff, image, kept, strip_rows, segments):
    _check(oracle, n, c, h, w, scale, L, k, coeff, image, kept, strip_rows, segments)


def _check_list(n, h, w, scale, entries, image, strip_rows=0, segments=0):
    wl = sr_synth.Workload("strips", 61, n, 3, h, w, scale, 72, 5, "f16", image)
    inp = sr_synth.make_inputs(wl, DEV)
    index, value = sr_synth.to_list(inp["coeff"], entries)
    out = [torch.full((n, 3, wl.H, wl.W), float("nan"), device=DEV, dtype=inp["lr"].dtype) for _ in range(2)]
    if strip_rows:
        _assert_strips(sr.sr_dict_assemble_list_walk(inp["lr"], index, value, inp["dict"], 72, 5, scale, 3, entries, out[0]), strip_rows, segments)
    for o, kernel in zip(out, (MFMA, GENERIC)):
        sr.sr_dict_assemble_list_ex(inp["lr"], index, value, inp["dict"], 72, 5, scale, 3, entries, o, kernel=kernel)
    got, want = out[0].float(), out[1].float()
    assert torch.isfinite(got).all()
    assert float((got - want).abs().max()) <= (5e-5 + (2.0 ** -10 if image == "f16" else 0.0)) * max(1.0, float(want.abs().max()))


@pytest.mark.parametrize("h, w, scale, entries, image", [(270, 480, 4, 8, "f32"), (301, 500, 3, 5, "f16"), (270, 477, 4, 16, "f32"), (301, 500, 3, 13, "f32")])
def test_strips_of_lists(h, w, scale, entries, image):
    _check_list(1, h, w, scale, entries, image)


@pytest.mark.parametrize("n, h, w, scale, entries, image, strip_rows, segments", [
    (1, 600, 800, 3, 8, "f32", 7, 1),
    (1, 601, 796, 3, 13, "f16", 7, 1),
    (2343, 2, 4, 3, 5, "f32", 6, 2),            # the register sets change hands between segments: an even and an odd number of rows
    (2400, 3, 4, 3, 13, "f32", 9, 2),
    (2251, 2, 3, 4, 8, "f16", 8, 2),
    (1030, 3, 34, 4, 16, "f32", 12, 2),
    (6200, 3, 4, 3, 8, "f32", 9, 3),
])
def test_strips_of_lists_as_launched(n, h, w, scale, entries, image, strip_rows, segments):
    _check_list(n, h, w, scale, entries, image, strip_rows, segments)


@pytest.mark.parametrize("h, w, scale, coeff", [(271, 473, 4, "f16"), (301, 501, 2, "bf16"), (333, 400, 3, "f16")])
def test_strips_of_logits(h, w, scale, coeff):
    """Same fp32 evaluation of the exponentials in both kernels (see test_gpu_logits.py)."""
    wl = sr_synth.Workload("strips", 62, 1, 3, h, w, scale, 72, 5, coeff, "f32")
    lr, z, d = sr_synth.make_lr(wl, DEV), sr_synth.make_logits(wl, DEV), sr_synth.make_dictionary(wl, DEV)
    out = [torch.full((1, 3, wl.H, wl.W), float("nan"), device=DEV) for _ in range(2)]
    for o, kernel in zip(out, (MFMA, GENERIC)):
        sr.sr_dict_assemble_ex(lr, z, d, 72, 5, scale, 3, o, opts=sr.make_options(kernel, coeff_kind=sr.SR_COEFF_LOGITS))
    assert torch.isfinite(out[0]).all()
    assert float((out[0] - out[1]).abs().max()) <= 5e-5


@pytest.mark.parametrize("n, c, h, L, coeff, image, kept", [
    (1, 1, 43, 72, "f16", "f32", None),
    (1, 1, 7, 72, "bf16", "f16", None),
    (1, 3, 43, 72, "f16", "f32", 30),                    # the forms and batches whose other sizes about this one take strips
    (1, 3, 43, 72, "bf16", "f32", 41),
    (1, 3, 43, 72, "f8", "f32", 30),
    (32, 3, 43, 72, "f16", "f32", None),
    (32, 3, 43, 72, "f8", "f32", None),
])
def test_one_column_more_than_a_strip(oracle, n, c, h, L, coeff, image, kept):
    """43 columns at x3 are 129: a last strip moved left to end at the edge would start at column 1 and look one column over the
    left edge, where the image is continued by copies of column 0 and the strip form has none there; both strips write the
    same pixels.  Such images take tiles."""
    wl = sr_synth.Workload("moved", 63, n, c, h, 43, 3, L, 5, coeff, image)
    inp = sr_synth.make_inputs(wl, DEV)
    inp["lr"][..., 0] = 1.0                               # a step at the left edge, where the two continuations differ most
    inp["lr"][..., 1:3] = 0.0
    rng = np.random.default_rng(h)
    lst = None if kept is None else rng.permutation(L)[:kept].astype(np.int32)
    gamma = None if kept is None else rng.uniform(0.5, 1.5, size=kept).astype(np.float32)
    check_full(oracle, wl, MFMA, kept=lst, gamma=gamma, inp=inp)


@pytest.mark.parametrize("coeff", ["f16", "bf16"])
def test_one_column_more_than_a_strip_logits(coeff):
    wl = sr_synth.Workload("moved", 64, 1, 3, 43, 43, 3, 72, 5, coeff, "f32")
    lr, z, d = sr_synth.make_lr(wl, DEV), sr_synth.make_logits(wl, DEV), sr_synth.make_dictionary(wl, DEV)
    lr[..., 0], lr[..., 1:3] = 1.0, 0.0
    out = [torch.full((1, 3, wl.H, wl.W), float("nan"), device=DEV) for _ in range(2)]
    for o, kernel in zip(out, (MFMA, GENERIC)):
        sr.sr_dict_assemble_ex(lr, z, d, 72, 5, 3, 3, o, opts=sr.make_options(kernel, coeff_kind=sr.SR_COEFF_LOGITS))
    assert torch.isfinite(out[0]).all()
    assert float((out[0] - out[1]).abs().max()) <= 5e-5


def _assert_tile(walk, width, rows):
    assert walk[0] == MFMA and walk[1][:3] == (1, width, rows), walk


@pytest.mark.parametrize("image", ["f32", "f16"])
def test_8_bit_tiles_where_strips_are_refused(oracle, image):
    """720 x 960 at x4: 128 x 24 tiles (30 rows of them, whole; 7.5 tiles wide)."""
    wl = sr_synth.Workload("tiles", 65, 1, 3, 180, 240, 4, 72, 5, "f8", image)
    inp = sr_synth.make_inputs(wl, DEV)
    out = torch.empty((1, 3, wl.H, wl.W), device=DEV, dtype=inp["lr"].dtype)
    _assert_tile(sr.sr_dict_assemble_walk(inp["lr"], inp["coeff"], inp["dict"], 72, 5, 4, 3, out), 128, 24)
    check_full(oracle, wl, MFMA, inp=inp)


@pytest.mark.parametrize("h, entries", [(180, 8), (178, 16)])
def test_list_strips_of_few_rows(h, entries):
    """1280 columns at x4: ten strips, segments of four rows; 712 rows are no whole number of them."""
    wl = sr_synth.Workload("tiles", 66, 1, 3, h, 320, 4, 72, 5, "f16", "f32")
    inp = sr_synth.make_inputs(wl, DEV)
    index, value = sr_synth.to_list(inp["coeff"], entries)
    out = [torch.full((1, 3, wl.H, wl.W), float("nan"), device=DEV) for _ in range(2)]
    assert sr.sr_dict_assemble_list_walk(inp["lr"], index, value, inp["dict"], 72, 5, 4, 3, entries, out[0])[1][0] == 2
    for o, kernel in zip(out, (MFMA, GENERIC)):
        sr.sr_dict_assemble_list_ex(inp["lr"], index, value, inp["dict"], 72, 5, 4, 3, entries, o, kernel=kernel)
    assert torch.isfinite(out[0]).all()
    assert float((out[0] - out[1]).abs().max()) <= 5e-5 * max(1.0, float(out[1].abs().max()))


@pytest.mark.parametrize("h, w, scale, L", [(16383, 16385, 2, 1), (25487, 4681, 3, 1)])
def test_images_of_just_below_4_gb(h, w, scale, L):
    """fp32 images that end 16 and 4 bytes below 4 GB: lanes outside them store nowhere, those inside everywhere."""
    n = h * scale * w * scale
    assert (1 << 32) - 4 * n in (16, 4)
    lr = torch.rand((1, 1, h, w), device=DEV)
    coeff = torch.randint(0x28, 0x40, (1, L, h * scale, w * scale), device=DEV, dtype=torch.uint8).view(torch.float8_e4m3fn)
    d = torch.randn((L, 5, 5), device=DEV) * 0.1
    guard = torch.full((n + 1024,), float("nan"), device=DEV)
    got = guard[:n].view(1, 1, h * scale, w * scale)
    want = torch.empty_like(got)
    for o, kernel in ((got, MFMA), (want, GENERIC)):
        sr.sr_dict_assemble_ex(lr, coeff, d, L, 5, scale, 1, o, opts=sr.make_options(kernel))
    assert torch.isnan(guard[n:]).all()
    worst = max(float((a - b).abs().max()) for a, b in zip(got[0, 0].split(2048), want[0, 0].split(2048)))
    assert worst <= 5e-5 * max(1.0, float(want.abs().max()))


# Rows that share 128-byte lines are read with ordinary loads from 400 thousand pixels on: a frame alone is below that (some run on the second matrix-core kernel then), in a batch it is not.  Every
# family of the rule, either form, rows off by 2 to 96 bytes, the last strip or tile moved left and not
@pytest.mark.parametrize("c, h, w, s, L, k, cd, kind", [
    (3, 100, 153, 4, 72, 5, "f16", "values"), (3, 130, 250, 2, 57, 5, "bf16", "values"), (3, 96, 168, 3, 72, 5, "f8", "values"), (1, 90, 202, 4, 72, 5, "f8", "values"),
    (3, 61, 151, 4, 72, 7, "f16", "values"), (1, 70, 141, 4, 128, 7, "bf16", "values"), (3, 101, 170, 3, 72, 5, "f16", "logits"), (3, 80, 130, 4, 66, 5, "bf16", "logits"),
    (3, 100, 150, 4, 128, 3, "f16", "values"), (3, 120, 209, 3, 128, 5, "f16", "values"),      # (on the second matrix-core kernel, in a batch too: the line between both)
    (3, 100, 150, 3, 72, 3, "f16", "values"), (3, 77, 104, 3, 128, 3, "bf16", "values"), (3, 120, 209, 2, 66, 3, "f8", "values"),
    (3, 77, 104, 2, 128, 5, "f16", "values"), (3, 90, 168, 4, 100, 5, "bf16", "values"), (3, 120, 209, 3, 90, 5, "f16", "values"), (1, 110, 201, 4, 50, 5, "f16", "values"), (3, 90, 141, 4, 30, 5, "f16", "values")])
def test_rows_that_share_lines_have_the_same_bits(c, h, w, s, L, k, cd, kind):
    wl = sr_synth.Workload("lines", 74, 2, c, h, w, s, L, k, cd, "f32", 0.0, 1.5)
    inp = sr_synth.make_inputs(wl, DEV)
    coeff = sr_synth.make_logits(wl, DEV) if kind == "logits" else inp["coeff"]
    assert wl.H * wl.W < 400_000 and wl.W * (1 if cd == "f8" else 2) % 128 != 0
    opts = sr.make_options(coeff_kind=sr.SR_COEFF_LOGITS if kind == "logits" else sr.SR_COEFF_VALUES)

    def run(n):
        pick = torch.arange(n, device=DEV) % 2
        out = torch.full((n, c, wl.H, wl.W), float("nan"), device=DEV)
        raw = coeff.view(torch.uint8) if cd == "f8" else coeff
        sr.sr_dict_assemble_ex(inp["lr"][pick].contiguous(), raw[pick].contiguous().view(coeff.dtype), inp["dict"], L, k, s, c, out, opts=opts)
        torch.cuda.synchronize()
        return out

    n = 2 * (1 + 1_100_000 // (wl.H * wl.W))         # two million pixels and more
    batch = [torch.empty((n, *t.shape[1:]), device=DEV, dtype=t.dtype) for t in (inp["lr"], coeff, torch.empty((1, c, wl.H, wl.W), device=DEV))]
    launched = sr.sr_dict_assemble_runs(batch[0], batch[1], inp["dict"], L, k, s, c, batch[2], opts=opts)[0]
    del batch
    assert launched == (sr.SR_RUNS_SLOTS if (w, L) in ((150, 128), (209, 128)) else sr.SR_RUNS_STREAMING)
    many = run(n)
    one = run(1)
    assert torch.isfinite(many).all() and torch.equal(many[0], one[0]) and torch.equal(many[-2], one[0]) and torch.equal(many[-1], many[1])
    if kind == "values":                             # (and the vector-ALU kernel agrees)
        gen = torch.empty_like(one)
        sr.sr_dict_assemble_ex(inp["lr"][:1], coeff[:1], inp["dict"], L, k, s, c, gen, opts=sr.make_options(sr.SR_KERNEL_GENERIC))
        assert float((gen - one).abs().max()) <= (1e-4 if cd == "bf16" else 5e-5) * max(1.0, float(gen.abs().max()))
