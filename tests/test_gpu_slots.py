"""Calls that no instantiation of the streaming matrix-core kernel holds (coefficients before the pixel-shuffle and logits in
most types and sizes): the library's own choice of kernel against the oracle, against the generic kernel over all the forms that
both take, and its distance from 64-bit arithmetic, which must not exceed the generic kernel's."""
import numpy as np
import pytest
import torch

import paper_2303_08999_amd as sr
import sr_synth
from test_gpu_parity import DEV, GENERIC, assert_parity, host, tolerance_ok
from test_gpu_logits import assert_logits_parity

pytestmark = pytest.mark.gpu
AUTO = sr.SR_KERNEL_AUTO


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    assert torch.cuda.is_available(), "these tests need the MI355X"
    sr.load()


def run(inp, wl, coeff, kernel, pre, logits, kept=None, gamma=None):
    out = torch.full((wl.n, wl.c, wl.H, wl.W), float("nan"), device=DEV, dtype=inp["lr"].dtype)
    opts = sr.make_options(kernel, 0, sr.SR_COEFF_PRE_SHUFFLE if pre else sr.SR_COEFF_PLANAR,
                           sr.SR_COEFF_LOGITS if logits else sr.SR_COEFF_VALUES)
    sr.sr_dict_assemble_ex(inp["lr"], coeff, inp["dict"], wl.L, wl.k, wl.scale, wl.c, out, kept=kept, gamma=gamma, opts=opts)
    torch.cuda.synchronize()
    return out


def runs(inp, wl, coeff, pre, logits, kept=None):
    """The kernel that AUTO launches, and its walk."""
    opts = sr.make_options(AUTO, 0, sr.SR_COEFF_PRE_SHUFFLE if pre else sr.SR_COEFF_PLANAR,
                           sr.SR_COEFF_LOGITS if logits else sr.SR_COEFF_VALUES)
    out = torch.empty((wl.n, wl.c, wl.H, wl.W), device=DEV, dtype=inp["lr"].dtype)
    return sr.sr_dict_assemble_runs(inp["lr"], coeff, inp["dict"], wl.L, wl.k, wl.scale, wl.c, out, kept=kept, opts=opts)


def make(wl, pre, logits):
    inp = sr_synth.make_inputs(wl, DEV)
    flat = sr_synth.make_logits(wl, DEV) if logits else inp["coeff"]
    return inp, flat, sr_synth.to_pre_shuffle(flat, wl.scale) if pre else flat


# words of one, two and four pixels at the end of rows that are no whole number of them; rows of one word; every scale, filter size,
# number of parts of the dictionary; capacities full and with one atom; one to three channels; both image types; kept lists
CASES = [
    # (N, C, h, w, scale, L, k, coeff, image, pre-shuffle, logits, kept)
    (1, 3, 9, 65, 2, 72, 5, "f16", "f32", True, False, None), (1, 1, 5, 33, 4, 128, 5, "f16", "f16", True, False, None),
    (2, 2, 7, 31, 3, 33, 7, "bf16", "f32", True, False, None), (1, 3, 11, 67, 3, 72, 5, "f8", "f32", True, False, None),
    (1, 1, 6, 130, 4, 40, 7, "f8", "f16", True, False, 17), (1, 3, 9, 35, 2, 100, 3, "f32", "f32", True, False, None),
    (1, 3, 4, 2, 4, 1, 5, "bf16", "f32", True, False, None), (1, 1, 3, 4, 2, 8, 3, "f8", "f32", True, False, None),
    (1, 3, 19, 61, 4, 72, 7, "f32", "f16", True, False, 30), (1, 2, 10, 1, 3, 16, 5, "f32", "f32", True, False, None),
    (1, 1, 13, 47, 3, 72, 5, "f16", "f32", False, True, None), (1, 3, 8, 25, 4, 128, 7, "bf16", "f16", False, True, None),
    (2, 3, 9, 50, 2, 50, 3, "f32", "f32", False, True, None), (1, 3, 6, 33, 4, 96, 5, "f16", "f32", True, True, None),
    (1, 1, 12, 29, 3, 72, 7, "f32", "f32", True, True, None), (1, 3, 7, 70, 2, 9, 5, "bf16", "f32", True, True, None),
    (1, 3, 11, 17, 3, 72, 7, "f8", "f32", False, False, 9), (1, 2, 30, 65, 2, 72, 5, "f8", "f32", False, False, None),
    (1, 3, 4, 2, 4, 17, 5, "bf16", "f32", True, False, None), (1, 1, 3, 4, 2, 15, 3, "f8", "f32", True, False, None),
    (1, 2, 10, 1, 3, 21, 5, "f32", "f32", True, False, None), (1, 3, 11, 17, 3, 72, 7, "f8", "f32", False, False, 33), (1, 3, 7, 70, 2, 12, 5, "bf16", "f32", True, True, None),
]
# those that are left to the generic kernel (the last five above are the same with as many atoms as this one takes)
FEW_ATOMS = [c for c in CASES if (c[5], c[6], c[7], c[11]) in ((1, 5, "bf16", None), (8, 3, "f8", None), (16, 5, "f32", None), (72, 7, "f8", 9), (9, 5, "bf16", None))]


@pytest.mark.parametrize("case", CASES, ids=lambda c: "N%dC%dh%dw%ds%dL%dk%d%s%s-%d%d-%s" % c)
def test_against_the_oracle(oracle, case):
    N, C, h, w, s, L, k, cd, io, pre, logits, nk = case
    wl = sr_synth.Workload("slots", 70, N, C, h, w, s, L, k, cd, io, 0.0, 1.5)
    inp, flat, coeff = make(wl, pre, logits)
    kept = gamma = None
    if nk:
        rng = np.random.default_rng(nk)
        kept = np.sort(rng.choice(L, size=nk, replace=False)).astype(np.int32)
        gamma = rng.uniform(0.5, 1.5, size=nk).astype(np.float32)
    assert runs(inp, wl, coeff, pre, logits, kept)[0] == (sr.SR_RUNS_GENERIC if case in FEW_ATOMS else sr.SR_RUNS_SLOTS)
    got = run(inp, wl, coeff, AUTO, pre, logits, kept, gamma)
    hi = host(inp)
    phi = oracle.softmax_logits(sr_synth.stored_numpy(flat)) if logits else sr_synth.stored_numpy(flat)
    ref = oracle.assemble(oracle.bicubic(hi["lr"], s), phi, hi["dict"], kept=kept, gamma=gamma)
    if logits:
        assert_logits_parity(got.float().cpu().numpy(), ref, io == "f16", case)
    else:
        # (fp32 bounds for every type: the dictionary's parts carry 22 bits and more)
        worst, tol, ok = tolerance_ok(got.float().cpu().numpy(), ref, "f16" if cd == "bf16" else cd, io == "f16")
        assert ok, (case, worst, tol)
    if io == "f32":
        # no further from 64-bit arithmetic than the generic kernel: both are a few roundings of fp32, so a tenth for chance
        gen = run(inp, wl, coeff, GENERIC, pre, logits, kept, gamma)
        rms = lambda x: float(np.sqrt(np.mean((x.double().cpu().numpy() - ref) ** 2)))
        assert rms(got) <= 1.1 * rms(gen) + 1e-9, (case, rms(got), rms(gen))


def test_random_shapes_against_the_generic_kernel():
    """Everything that both take: orders, types, sizes, kept lists, batches."""
    rng = np.random.default_rng(11)
    compared = 0
    for index in range(260):
        pre, logits = bool(rng.integers(2)), bool(rng.integers(2))
        cd = str(rng.choice(["f16", "bf16", "f32"] if logits else ["f16", "bf16", "f32", "f8"]))
        k, s, C, N = int(rng.choice([3, 5, 7])), int(rng.choice([2, 3, 4])), int(rng.choice([1, 2, 3])), int(rng.choice([1, 1, 2, 5]))
        L = int(rng.choice([72, 128, int(rng.integers(1, 129))]))
        big = index % 10 == 0
        h, w = int(rng.integers(1, 160 if big else 30)), int(rng.integers(1, 300 if big else 80))
        if N * h * w * s * s * L > 60e6:
            continue
        wl = sr_synth.Workload("slotsr", 700 + index, N, C, h, w, s, L, k, cd, str(rng.choice(["f32", "f16"])), 0.0, 1.5)
        inp, flat, coeff = make(wl, pre, logits)
        kept = gamma = None
        if not logits and rng.random() < 0.4:
            nk = int(rng.integers(1, L + 1))
            kept = np.sort(rng.choice(L, size=nk, replace=False)).astype(np.int32)
            gamma = rng.uniform(0.5, 1.5, size=nk).astype(np.float32)
        if runs(inp, wl, coeff, pre, logits, kept)[0] != sr.SR_RUNS_SLOTS:
            continue
        a = run(inp, wl, coeff, AUTO, pre, logits, kept, gamma).float()
        b = run(inp, wl, coeff, GENERIC, pre, logits, kept, gamma).float()
        what = (wl, pre, logits, kept)
        assert torch.isfinite(a).all(), what
        # fp32 rounding order, half a step of an fp16 image; logits: an exponential next to a tie may round the other way on one side
        # (planar bfloat16 calls of the streaming kernel have its dictionary of 16 bits, see parity_bound)
        tol = (2.5e-4 if logits else 1e-4 if cd == "bf16" else 5e-5) + (2.0 ** -10 if wl.lr_dtype == "f16" else 0.0)
        err = float((a - b).abs().max())
        assert err <= tol * max(1.0, float(b.abs().max())), (what, err)
        compared += 1
    assert compared >= 150, compared


# Planar coefficients that the streaming kernel has an instantiation for and that go here all the same, and their neighbours on the
# other side of each line: the result is the matrix-core kernel's either way
@pytest.mark.parametrize("n, c, h, w, s, L, k, cd, io, slots", [
    (1, 3, 60, 70, 3, 100, 5, "f8", "f32", True), (1, 1, 3, 5, 2, 128, 3, "f32", "f16", True), (2, 1, 40, 25, 4, 73, 5, "f32", "f32", True),
    (1, 3, 82, 155, 2, 72, 7, "f8", "f32", True), (1, 3, 250, 260, 2, 72, 7, "f8", "f32", True), (1, 1, 64, 64, 2, 72, 5, "f32", "f32", True),
    (1, 1, 100, 110, 2, 72, 5, "f32", "f32", False), (1, 3, 93, 187, 3, 50, 5, "f32", "f16", True), (1, 3, 90, 120, 4, 72, 5, "f32", "f32", True), (1, 3, 90, 120, 4, 48, 5, "f32", "f32", False), (1, 1, 173, 352, 2, 115, 3, "f32", "f16", False),
    (1, 1, 3000, 4, 4, 98, 5, "f32", "f16", True), (1, 3, 60, 140, 4, 30, 7, "f32", "f32", True), (1, 3, 170, 175, 4, 128, 5, "bf16", "f16", False),
    (1, 3, 125, 131, 2, 128, 3, "f16", "f32", True), (1, 3, 150, 311, 3, 72, 3, "f16", "f32", True), (1, 3, 150, 320, 3, 72, 3, "f16", "f32", False), (1, 3, 150, 311, 3, 72, 5, "f16", "f32", False),
    (1, 1, 109, 152, 3, 72, 5, "f16", "f16", True), (1, 3, 300, 301, 3, 128, 5, "bf16", "f32", True), (1, 3, 10, 56, 2, 72, 3, "f16", "f32", True), (1, 3, 10, 40, 2, 72, 5, "f16", "f32", False)])
def test_planar_calls_that_are_faster_here(oracle, n, c, h, w, s, L, k, cd, io, slots):
    wl = sr_synth.Workload("slotsp", 72, n, c, h, w, s, L, k, cd, io, 0.0, 1.5)
    inp = sr_synth.make_inputs(wl, DEV)
    assert runs(inp, wl, inp["coeff"], False, False)[0] == (sr.SR_RUNS_SLOTS if slots else sr.SR_RUNS_STREAMING)
    got = run(inp, wl, inp["coeff"], sr.SR_KERNEL_MFMA, False, False)
    gen = run(inp, wl, inp["coeff"], GENERIC, False, False)
    assert torch.isfinite(got).all()
    tol = (5e-5 if cd != "bf16" else 1e-4) + (2.0 ** -10 if io == "f16" else 0.0)
    assert float((got.float() - gen.float()).abs().max()) <= tol * max(1.0, float(gen.float().abs().max()))
    if n == 1 and wl.H * wl.W * L < 30e6:
        hi = host(inp)
        ref = oracle.assemble(oracle.bicubic(hi["lr"], s), sr_synth.stored_numpy(inp["coeff"]), hi["dict"])
        worst, t, ok = tolerance_ok(got.float().cpu().numpy(), ref, cd, io == "f16")
        assert ok, (worst, t)


def test_an_infinite_image_value_stays_within_its_patches():
    """The halves of a filter have unequal numbers of rows: the one that pads the second must not reach beyond the patch."""
    wl = sr_synth.Workload("slotsi", 71, 1, 1, 12, 40, 2, 72, 5, "f32", "f32", 0.0, 1.5)
    inp, flat, coeff = make(wl, True, False)
    inp["lr"][0, 0, 6, 20] = float("inf")
    a, b = (run(inp, wl, coeff, kernel, True, False) for kernel in (AUTO, GENERIC))
    assert torch.equal(torch.isfinite(a), torch.isfinite(b)) and not torch.isfinite(b).all()


# More tiles than workgroups, tiles of one or two rows, and a last tile of a row with fewer units than a workgroup has wavefronts: those
# that sit it out still have to fetch their first unit of the next tile
@pytest.mark.parametrize("n, c, h, w, s, L, k, cd, logits", [
    (1, 1, 104, 69, 4, 128, 5, "f32", False), (1, 3, 119, 135, 4, 100, 3, "f32", False), (1, 2, 164, 143, 4, 128, 7, "f32", False),
    (1, 2, 280, 611, 2, 128, 7, "f32", False), (1, 1, 123, 289, 2, 56, 7, "f32", False), (4, 2, 131, 321, 2, 100, 3, "f32", False),
    (1, 1, 172, 129, 2, 73, 5, "f32", False), (400, 1, 1, 260, 2, 72, 5, "f32", True), (400, 2, 1, 260, 2, 40, 5, "f16", True),
    (1, 1, 219, 402, 2, 72, 3, "bf16", True), (1, 1, 146, 575, 3, 55, 3, "f16", True)])
def test_wavefronts_without_a_unit_in_a_partial_tile(n, c, h, w, s, L, k, cd, logits):
    wl = sr_synth.Workload("slotst", 73, n, c, h, w, s, L, k, cd, "f32", 0.0, 1.5)
    inp, flat, coeff = make(wl, False, logits)
    kernel, (form, width, rows, tiles, workgroups, waves) = runs(inp, wl, coeff, False, logits)
    units = rows * -(-(wl.W % width) // (32 if cd == "f32" else 64))         # of a partial tile
    assert kernel == sr.SR_RUNS_SLOTS and tiles > workgroups and 0 < units < waves
    got = run(inp, wl, coeff, AUTO, False, logits)
    gen = run(inp, wl, coeff, GENERIC, False, logits)
    assert torch.isfinite(got).all()
    tol = 2.5e-4 if logits else (5e-5 if cd != "bf16" else 1e-4)
    assert float((got - gen).abs().max()) <= tol * max(1.0, float(gen.abs().max()))


# A planar call gives the streaming kernel's bits whichever kernel it is sent to: the frames of a batch one by one and together
@pytest.mark.parametrize("k, c, L, cd, io", [(3, 1, 72, "f16", "f32"), (3, 1, 40, "bf16", "f32"), (5, 1, 72, "f16", "f16"), (5, 1, 128, "bf16", "f32"),
                                             (7, 1, 100, "f16", "f32"), (7, 1, 30, "bf16", "f32"), (5, 3, 72, "f32", "f32"), (7, 1, 72, "f32", "f16")])
def test_frames_of_a_batch_have_the_bits_of_single_ones(k, c, L, cd, io):
    n = 170
    wl = sr_synth.Workload("slotsb", 74, n, c, 24, 64, 2, L, k, cd, io, 0.0, 1.5)
    one = sr_synth.Workload("slotsb", 74, 1, c, 24, 64, 2, L, k, cd, io, 0.0, 1.5)
    inp = sr_synth.make_inputs(wl, DEV)
    assert runs(inp, wl, inp["coeff"], False, False)[0] == sr.SR_RUNS_STREAMING
    batch = run(inp, wl, inp["coeff"], AUTO, False, False)
    for i in (0, n // 2, n - 1):
        single = dict(inp, lr=inp["lr"][i:i + 1].contiguous())
        coeff = inp["coeff"][i:i + 1].contiguous()
        assert runs(single, one, coeff, False, False)[0] == sr.SR_RUNS_SLOTS
        assert torch.equal(run(single, one, coeff, AUTO, False, False), batch[i:i + 1])


# The dictionary's 16-bit parts: a power of two goes through every form without a trace, and small atoms beside large ones keep their bits
FORMS = [(3, 72, 5, "f16", True, False), (1, 40, 3, "f8", True, False), (1, 128, 7, "bf16", True, False), (3, 100, 5, "f32", True, False),
         (3, 72, 3, "f16", False, True), (1, 100, 5, "bf16", False, True), (2, 30, 7, "f32", True, True), (2, 72, 5, "f8", False, False)]


@pytest.mark.parametrize("c, L, k, cd, pre, logits", FORMS)
@pytest.mark.parametrize("power", [20, 60, -22, -60])
def test_dictionaries_of_any_magnitude(c, L, k, cd, pre, logits, power):
    wl = sr_synth.Workload("slotsm", 75, 1, c, 15, 67, 2, L, k, cd, "f32", 0.0, 1.5)
    inp, flat, coeff = make(wl, pre, logits)
    assert runs(inp, wl, coeff, pre, logits)[0] == sr.SR_RUNS_SLOTS
    ref = run(inp, wl, coeff, AUTO, pre, logits)
    got = run(dict(inp, dict=inp["dict"] * 2.0 ** power), wl, coeff, AUTO, pre, logits)
    assert torch.equal(got, ref * 2.0 ** power)
    if not logits:                                  # the same as a scale of the kept atoms
        kept, gamma = np.arange(L, dtype=np.int32), np.full(L, 2.0 ** power, np.float32)
        assert torch.equal(run(inp, wl, coeff, AUTO, pre, logits, kept, gamma), got)


@pytest.mark.parametrize("c, L, k, cd, pre, logits", FORMS)
def test_small_atoms_beside_large_ones(c, L, k, cd, pre, logits):
    """Only the last atom, of entries around 1e-7 of the others', takes part: 22 bits of it and more are asked for, i.e. what the bound of
    fp32 sums leaves."""
    wl = sr_synth.Workload("slotsm", 76, 1, c, 15, 67, 2, L, k, cd, "f32", 0.0, 1.5)
    inp, flat, coeff = make(wl, pre, logits)
    only = torch.full(flat.shape, -float("inf") if logits else 0.0, device=DEV)
    only[:, L - 1] = 1.0
    flat = only.to(flat.dtype)
    coeff = sr_synth.to_pre_shuffle(flat, wl.scale) if pre else flat
    inp["dict"][..., L - 1, :, :] *= 1e-7
    got, gen = (run(inp, wl, coeff, kernel, pre, logits) for kernel in (AUTO, GENERIC))
    # (k^2 products of an entry that is off by 2^-23 of itself at most, sums of them in another order)
    assert float((got - gen).abs().max()) <= 2e-6 * float(gen.abs().max())


@pytest.mark.parametrize("c, L, k, cd, pre, logits", FORMS + [(1, 72, 5, "f16", True, False), (3, 17, 7, "bf16", True, False), (2, 72, 5, "f32", False, False),
                                                              (1, 72, 7, "f32", False, True), (3, 128, 3, "f8", True, False)])
@pytest.mark.parametrize("io", ["f32", "f16"])
def test_infinities_and_nan_as_in_the_generic_kernel(c, L, k, cd, pre, logits, io):
    wl = sr_synth.Workload("slotsn", 77, 2, c, 14, 71, 3, L, k, cd, io, 0.0, 1.5)
    inp, flat, coeff = make(wl, pre, logits)
    assert runs(inp, wl, coeff, pre, logits)[0] == sr.SR_RUNS_SLOTS
    inf, nan = float("inf"), float("nan")
    changed = flat.float()
    values = [-inf] if logits else [inf, -inf, nan] if cd != "f8" else [nan]
    if cd == "bf16" and logits:
        values += [-1e37, -3e38]
    for i in range(60):                             # the first and the last atom, and any; edges of rows and units, and any
        atom = (0, L - 1, (7 * i) % L)[i % 3]
        y, x = ((0, 0), (wl.H - 1, wl.W - 1), ((11 * i) % wl.H, (37 * i) % wl.W))[(i // 3) % 3]
        changed[i % 2, atom, y, x] = values[(i // 2) % len(values)]
    if logits:
        changed[0, :, 5, 6] = -inf                  # no atom is left
    changed = changed.to(flat.dtype)
    changed = sr_synth.to_pre_shuffle(changed, wl.scale) if pre else changed
    image, entry = inp["lr"].clone(), inp["dict"].clone()
    image[1, c - 1, 6, 20], image[0, 0, 0, 0], image[0, 0, 13, 70] = inf, -inf, nan
    entry[..., L // 2, k // 2, 0] = inf
    for what, other, phi in (("coefficients", inp, changed), ("image", dict(inp, lr=image), coeff), ("dictionary", dict(inp, dict=entry), coeff)):
        got, gen = (run(other, wl, phi, kernel, pre, logits).float() for kernel in (AUTO, GENERIC))
        odd = ~torch.isfinite(gen)
        assert odd.any() or (logits and what == "coefficients"), what
        assert torch.equal(torch.isfinite(got), ~odd), what
        assert torch.equal(torch.nan_to_num(got[odd], 7.0), torch.nan_to_num(gen[odd], 7.0)), what
        tol = (2.5e-4 if logits else 5e-5) + (2.0 ** -10 if io == "f16" else 0.0)
        assert not (~odd).any() or float((got - gen)[~odd].abs().max()) <= tol * max(1.0, float(gen[~odd].abs().max())), what


# 5x5 atoms of three channels in 16 bits, the commonest calls: a small frame alone runs here, in a batch on the streaming kernel (in tiles or strips); capacities
# 32 and 72 at their edges, ragged rows, narrow images, one row of tiles
@pytest.mark.parametrize("h, w, s, L, kept, cd, io", [
    (40, 56, 2, 72, None, "f16", "f32"), (45, 47, 3, 72, None, "bf16", "f16"), (56, 85, 3, 72, None, "f16", "f32"), (12, 60, 4, 72, None, "f16", "f16"),
    (130, 253, 3, 33, None, "bf16", "f32"), (29, 44, 3, 65, None, "f16", "f32"), (61, 68, 2, 72, 50, "f16", "f32"), (250, 300, 2, 32, None, "bf16", "f32"),
    (141, 237, 3, 72, 17, "f16", "f16"), (122, 163, 4, 72, None, "f16", "f32"), (216, 306, 2, 48, None, "bf16", "f32")])
def test_a_small_frame_has_the_bits_it_has_in_a_batch(oracle, h, w, s, L, kept, cd, io):
    wl = sr_synth.Workload("slotsb", 73, 2, 3, h, w, s, L, 5, cd, io, 0.0, 1.5)
    inp = sr_synth.make_inputs(wl, DEV)
    atoms = None if kept is None else np.sort(np.random.default_rng(L).choice(L, size=kept, replace=False)).astype(np.int32)
    gamma = None if kept is None else np.linspace(0.5, 1.5, kept).astype(np.float32)
    n = 2 + 2_000_000 // (wl.H * wl.W)
    many = sr_synth.Workload("slotsb", 73, n, 3, h, w, s, L, 5, cd, io, 0.0, 1.5)
    batch = {"lr": inp["lr"][torch.arange(n, device=DEV) % 2].contiguous(), "dict": inp["dict"]}
    coeff = inp["coeff"][torch.arange(n, device=DEV) % 2].contiguous()
    assert runs(batch, many, coeff, False, False, atoms)[0] == sr.SR_RUNS_STREAMING
    together = run(batch, many, coeff, AUTO, False, False, atoms, gamma)
    for b in range(2):
        one = sr_synth.Workload("slotsb", 73, 1, 3, h, w, s, L, 5, cd, io, 0.0, 1.5)
        alone = {"lr": inp["lr"][b:b + 1].contiguous(), "dict": inp["dict"]}
        assert runs(alone, one, inp["coeff"][b:b + 1], False, False, atoms)[0] == sr.SR_RUNS_SLOTS
        assert torch.equal(run(alone, one, inp["coeff"][b:b + 1].contiguous(), AUTO, False, False, atoms, gamma)[0], together[b])
        assert torch.equal(together[b + n // 2 * 2 - 2], together[b])
        # (and both are what the oracle gives: the streaming kernel's small, ragged frames too)
        ref = oracle.dict_assemble(alone["lr"].cpu().numpy(), sr_synth.stored_numpy(inp["coeff"][b:b + 1].contiguous()), inp["dict"].cpu().numpy(), s, kept=atoms, gamma=gamma)
        assert_parity(together[b:b + 1].float().cpu().numpy(), ref, cd, io == "f16", "in a batch")


@pytest.mark.parametrize("h, w, s, L, cd, io, pre", [
    (40, 56, 2, 72, "f16", "f32", False), (45, 47, 3, 72, "bf16", "f16", False), (30, 60, 4, 66, "f16", "f16", True), (41, 66, 2, 72, "f16", "f32", True),
    (20, 33, 4, 72, "f16", "f32", True), (29, 44, 3, 72, "bf16", "f32", True)])
def test_small_frames_of_element_aligned_tensors_and_values_beyond_fp16(h, w, s, L, cd, io, pre):
    """Tensors that start one element into their allocation, and a dictionary or a coefficient outside fp16 or not finite: what the same frame has in aligned tensors, and
    in a batch (which the streaming kernel serves where the LR width is a multiple of 4 or the order is planar)."""
    wl = sr_synth.Workload("slotsa", 75, 1, 3, h, w, s, L, 5, cd, io, 0.0, 1.5)
    inp = sr_synth.make_inputs(wl, DEV)
    coeff = sr_synth.to_pre_shuffle(inp["coeff"], s) if pre else inp["coeff"]
    assert runs(inp, wl, coeff, pre, False)[0] == sr.SR_RUNS_SLOTS

    def shifted(t):
        return torch.zeros(t.numel() + 1, device=DEV, dtype=t.dtype)[1:].view(t.shape).copy_(t)

    moved = {"lr": shifted(inp["lr"]), "dict": shifted(inp["dict"])}
    assert torch.equal(run(moved, wl, shifted(coeff), AUTO, pre, False), run(inp, wl, coeff, AUTO, pre, False))
    n = 1 + 3_500_000 // (wl.H * wl.W)
    many = sr_synth.Workload("slotsa", 75, n, 3, h, w, s, L, 5, cd, io, 0.0, 1.5)
    for what in ("dictionary", "inf", "nan"):
        one, c = dict(inp), coeff.clone()
        if what == "dictionary":
            one["dict"] = inp["dict"].clone()
            one["dict"].view(L, 25)[3] = 1e5
        else:
            c.view(-1)[c.numel() // 2 + 7] = float(what)
        batch = {"lr": inp["lr"].expand(n, -1, -1, -1).contiguous(), "dict": one["dict"]}
        cs = c.expand(n, -1, -1, -1).contiguous()
        if not pre or (s != 3 and w % 4 == 0):
            assert runs(batch, many, cs, pre, False)[0] == sr.SR_RUNS_STREAMING
        alone, together = run(one, wl, c, AUTO, pre, False), run(batch, many, cs, AUTO, pre, False)
        assert torch.equal(torch.nan_to_num(alone[0], 7.0, 8.0, 9.0), torch.nan_to_num(together[n // 2], 7.0, 8.0, 9.0)), what
