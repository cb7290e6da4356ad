"""GPU parity of the selection's normal equations (sr_atom_gram) against the numpy
oracle, and the whole chain on a planted problem: up-sample, normal equations, Alg. 1,
selective assembly with the kept list and gamma it returned."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
import paper_2303_08999_amd as sr
import sr_synth
from oracle import select_oracle as so

pytestmark = pytest.mark.gpu
DEV = "cuda"

CASES = [
    # (N, C, h, w, scale, L, k, coeff dtype, stride)
    (1, 3, 9, 11, 2, 5, 3, "f32", 1),
    (2, 3, 12, 17, 4, 72, 5, "f16", 1),      # 3264 lattice pixels: 51 runs of 64 samples
    (1, 1, 16, 16, 3, 128, 7, "f16", 2),     # the largest atom count: 9 column blocks, 12 blocks per wavefront
    (3, 2, 10, 13, 2, 17, 7, "f32", 3),      # ragged lattice, L + 1 not a multiple of 4
    (1, 3, 40, 48, 4, 72, 5, "f16", 5),
    (1, 16, 6, 7, 2, 3, 3, "f32", 1),        # 16 channels
    (2, 3, 11, 14, 4, 40, 5, "f8", 2),       # coefficients stored as 8-bit E4M3
    (1, 3, 40, 50, 4, 72, 5, "bf16", 1),     # ... as bfloat16, several runs per workgroup
    # more runs than workgroups, so that every workgroup walks several runs and channels
    (1, 3, 64, 80, 4, 72, 5, "f16", 1),      # 1280 runs of one lattice row segment each
    (1, 1, 96, 100, 4, 20, 5, "f32", 1),     # one channel: a new run every iteration, 2688 runs
    (2, 2, 120, 130, 3, 72, 3, "f8", 2),     # two channels, two images, ragged last segment
    (1, 3, 30, 500, 2, 100, 7, "f16", 4),    # 7 x 7, 9 column blocks, stride 4: long staged segments
]


def _inputs(case):
    N, C, h, w, s, L, k, cd, stride = case
    wl = sr_synth.Workload("gram", 30, N, C, h, w, s, L, k, cd, "f32", 0.0, 1.5)
    inp = sr_synth.make_inputs(wl, DEV)
    up = torch.empty((N, C, wl.H, wl.W), device=DEV)
    sr.sr_bicubic_upsample(inp["lr"], s, C, up)
    g = torch.Generator(device=DEV).manual_seed(77 + L)
    target = torch.rand((N, C, wl.H, wl.W), device=DEV, generator=g)
    return wl, inp, up, target


@pytest.mark.parametrize("case", CASES, ids=lambda c: "N%dC%dh%dw%ds%dL%dk%d%sst%d" % c)
def test_normal_equations_match_the_oracle(oracle, case):
    wl, inp, up, target = _inputs(case)
    stride = case[-1]
    normal = sr.sr_atom_gram(up, inp["coeff"], inp["dict"], target, wl.L, wl.k, wl.c, stride)
    again = sr.sr_atom_gram(up, inp["coeff"], inp["dict"], target, wl.L, wl.k, wl.c, stride)
    torch.cuda.synchronize()
    assert torch.equal(normal, again), "the sums must not depend on the run"
    got = normal.cpu().numpy()
    L = wl.L
    G, b, hh, M = got[:L * L].reshape(L, L), got[L * L:L * L + L], got[L * L + L], got[L * L + L + 1]
    U = oracle.bicubic(inp["lr"].cpu().numpy(), wl.scale)
    G0, b0, hh0, M0 = so.normal_equations(U, sr_synth.stored_numpy(inp["coeff"]), inp["dict"].cpu().numpy(),
                                          target.cpu().numpy(), stride)
    assert M == M0
    assert np.array_equal(G, G.T)
    # fp32 responses (relative 1e-6 each), fp32 sums over 64 samples, double beyond
    scale = np.sqrt(np.outer(np.diag(G0), np.diag(G0)))
    assert np.abs(G - G0).max() <= 2e-5 * scale.max() and (np.abs(G - G0) <= 2e-5 * scale + 1e-12).all()
    assert (np.abs(b - b0) <= 2e-5 * np.sqrt(np.diag(G0) * hh0) + 1e-12).all()
    assert abs(hh - hh0) <= 1e-6 * hh0


def test_normal_equations_on_random_shapes(oracle):
    """Sixty seeded shapes over both kernel forms: every stride from 1 to 7, one to sixteen
    channels, all four coefficient types, atom counts around every block boundary."""
    rng = np.random.default_rng(5)
    done = 0
    while done < 60:
        k = int(rng.choice([3, 5, 5, 7]))
        s = int(rng.choice([2, 3, 4]))
        C = int(rng.choice([1, 1, 2, 3, 3, 4, 7, 16]))
        N = int(rng.choice([1, 1, 2, 3]))
        cd = str(rng.choice(["f16", "bf16", "f32", "f8"]))
        L = int(rng.choice([int(rng.integers(1, 129)), 72, 16, 31, 32, 33, 79, 80, 81, 128]))
        stride = int(rng.choice([1, 1, 2, 3, 4, 5, 7]))
        h, w = int(rng.integers(2, 60)), int(rng.integers(2, 120))
        if L * C * h * w * s * s * N > 40e6:
            continue
        done += 1
        wl = sr_synth.Workload("gramr", 300 + done, N, C, h, w, s, L, k, cd, "f32", 0.0, 1.5)
        inp = sr_synth.make_inputs(wl, DEV)
        up = torch.empty((N, C, wl.H, wl.W), device=DEV)
        sr.sr_bicubic_upsample(inp["lr"], s, C, up)
        g = torch.Generator(device=DEV).manual_seed(77 + done)
        target = torch.rand((N, C, wl.H, wl.W), device=DEV, generator=g)
        got = sr.sr_atom_gram(up, inp["coeff"], inp["dict"], target, L, k, C, stride).cpu().numpy()
        G, b, hh, M = got[:L * L].reshape(L, L), got[L * L:L * L + L], got[L * L + L], got[L * L + L + 1]
        G0, b0, hh0, M0 = so.normal_equations(up.cpu().numpy().astype(np.float64), sr_synth.stored_numpy(inp["coeff"]),
                                              inp["dict"].cpu().numpy(), target.cpu().numpy(), stride)
        case = (N, C, h, w, s, L, k, cd, stride)
        scale = np.sqrt(np.outer(np.diag(G0), np.diag(G0)))
        assert M == M0 and np.array_equal(G, G.T), case
        assert np.abs(G - G0).max() <= 2e-5 * scale.max() and (np.abs(G - G0) <= 2e-5 * scale + 1e-12).all(), case
        assert (np.abs(b - b0) <= 2e-5 * np.sqrt(np.diag(G0) * hh0) + 1e-12).all(), case
        assert abs(hh - hh0) <= 1e-6 * hh0, case


# The form that keeps the whole triangle in a wavefront's registers: the last item of a row with 1, 15, 16 and 17 samples, rows
# that start on odd elements (four coefficients are one load), every number of column blocks, fewer items than wavefronts
# and several per wavefront, a stride that leaves one sample
@pytest.mark.parametrize("N,C,h,w,s,L,k,cd,stride", [
    (1, 1, 8, 8, 2, 72, 5, "f16", 16), (1, 3, 9, 11, 3, 79, 5, "bf16", 2), (1, 1, 13, 31, 3, 63, 3, "f8", 1), (2, 3, 40, 37, 3, 15, 7, "f16", 1),
    (1, 2, 60, 49, 3, 47, 5, "f32", 3), (1, 3, 50, 83, 3, 72, 5, "f8", 1), (1, 4, 33, 17, 4, 72, 7, "f16", 4),
    (1, 1, 20, 33, 2, 16, 5, "f16", 1), (1, 3, 21, 30, 2, 64, 3, "f32", 2)])          # the last block holds the target only
def test_triangle_in_registers(N, C, h, w, s, L, k, cd, stride):
    wl, inp, up, target = _inputs((N, C, h, w, s, L, k, cd, stride))
    got = sr.sr_atom_gram(up, inp["coeff"], inp["dict"], target, L, k, C, stride).cpu().numpy()
    G0, b0, hh0, M0 = so.normal_equations(up.cpu().numpy().astype(np.float64), sr_synth.stored_numpy(inp["coeff"]),
                                          inp["dict"].cpu().numpy(), target.cpu().numpy(), stride)
    ref = np.concatenate([G0.reshape(-1), b0, [hh0, M0]])
    # fp32 responses of k^2 products (2^-24 each, partial sums a few times the result) and fp32 sums over at most 64 samples
    tol = 1e-5 * np.sqrt(np.concatenate([np.outer(np.diag(G0), np.diag(G0)).reshape(-1), np.diag(G0) * hh0, [hh0 ** 2, M0 ** 2]]))
    assert (np.abs(got - ref) <= tol + 1e-12).all()
    if cd in ("f16", "f32"):                        # what is not a number stays within its atom
        inp["coeff"][0, L - 1, 0, 0] = float("nan")
        bad = sr.sr_atom_gram(up, inp["coeff"], inp["dict"], target, L, k, C, stride).cpu().numpy()
        mine = np.zeros((L, L), bool)
        mine[L - 1], mine[:, L - 1] = True, True
        mine = np.concatenate([mine.reshape(-1), np.arange(L) == L - 1, [False, False]])
        assert np.isnan(bad[mine]).all() and np.array_equal(bad[~mine], got[~mine])


def test_empty_batch_and_undersized_scratch():
    wl, inp, up, target = _inputs(CASES[0])
    z = torch.empty((0, 3, wl.H, wl.W), device=DEV)
    zc = torch.empty((0, wl.L, wl.H, wl.W), device=DEV)
    normal = sr.sr_atom_gram(z, zc, inp["dict"], z.clone(), wl.L, wl.k, 3)
    torch.cuda.synchronize()
    assert not normal.cpu().numpy().any()
    small = torch.empty(1024, device=DEV, dtype=torch.uint8)
    with pytest.raises(sr.SrError) as err:
        sr.sr_atom_gram(up, inp["coeff"], inp["dict"], target, wl.L, wl.k, 3, workspace=small)
    assert err.value.status == -2


# Planes of 2^26 fp32, 2^27 16-bit and 2^28 8-bit elements and more: 16 of them pass 4 GB; and of 2^30, whose patch operands do
@pytest.mark.parametrize("c, h, w, L, k, cd, stride", [(2, 8192, 8192, 18, 5, torch.float32, 61), (1, 8192, 8201, 2, 3, torch.float32, 1),
                                                       (2, 11600, 11603, 16, 7, torch.float16, 53), (1, 32768, 32771, 2, 3, torch.float8_e4m3fn, 127)])
def test_planes_beyond_32_bit_offsets(c, h, w, L, k, cd, stride):
    g = torch.Generator(device=DEV)
    g.manual_seed(78)
    up, target = (torch.rand((1, c, h, w), generator=g, device=DEV) for _ in range(2))
    coeff = torch.empty((1, L, h, w), device=DEV, dtype=cd)
    for l in range(L):
        coeff[0, l] = torch.rand((h, w), generator=g, device=DEV).to(cd)
    d = torch.rand((L, k, k), generator=g, device=DEV)
    got = sr.sr_atom_gram(up, coeff, d, target, L, k, c, stride).cpu().numpy()
    ref = torch.zeros((L + 1, L + 1), device=DEV, dtype=torch.float64)
    xs, r = torch.arange(0, w, stride, device=DEV), (k - 1) // 2
    for ys in torch.arange(0, h, stride, device=DEV).split(64):
        phi = coeff[0, :, ys][:, :, xs].double().reshape(L, -1) if cd != torch.float8_e4m3fn else torch.stack(
            [coeff[0, l].view(torch.uint8)[ys][:, xs].view(cd).double().reshape(-1) for l in range(L)])
        for ch in range(c):
            taps = [up[0, ch][(ys + i // k - r).clamp(0, h - 1)][:, (xs + i % k - r).clamp(0, w - 1)].double().reshape(-1) for i in range(k * k)]
            resp = torch.cat([(d.reshape(L, -1).double() @ torch.stack(taps)) * phi, target[0, ch][ys][:, xs].double().reshape(1, -1)])
            ref += resp @ resp.T.contiguous()
    ref = ref.cpu().numpy()
    G, b, hh = got[:L * L].reshape(L, L), got[L * L:L * L + L], got[L * L + L]
    assert got[-1] == c * len(range(0, h, stride)) * len(range(0, w, stride))
    size = np.sqrt(np.diag(ref))                    # (the bound of test_triangle_in_registers)
    assert (np.abs(G - ref[:L, :L]) <= 1e-5 * np.outer(size[:L], size[:L])).all()
    assert (np.abs(b - ref[:L, L]) <= 1e-5 * size[:L] * size[L]).all() and abs(hh - ref[L, L]) <= 1e-5 * ref[L, L]


@pytest.mark.parametrize("n, h, w, L", [(0, 8, 8, 72), (3, 0, 40, 72), (2, 40, 0, 15), (1, 0, 0, 100)])
@pytest.mark.parametrize("cd", [sr.SR_F16, sr.SR_F32])
def test_empty_images_read_nothing(n, h, w, L, cd):
    """An empty call need not bring any tensor: the normal equations are zero, and no kernel looks at a pointer."""
    shapes = [(sr.SR_F32, n, 3, h, w), (cd, n, L, h, w), (sr.SR_F32, 1, L, 5, 5), (sr.SR_F32, n, 3, h, w)]
    up, coeff, d, target = [sr.sr_tensor(None, *s) for s in shapes]
    size = sr.sr_atom_gram_workspace_bytes(L)
    workspace = torch.full((size // 8,), float("nan"), device=DEV, dtype=torch.float64)
    normal = torch.full((L * L + L + 2,), float("nan"), device=DEV, dtype=torch.float64)
    assert sr.load().sr_atom_gram(up, coeff, d, target, L, 5, 3, 1, workspace.data_ptr(), size, normal.data_ptr(), 0) == 0
    torch.cuda.synchronize()
    assert not normal.cpu().numpy().any()


def test_whole_chain_recovers_a_planted_selection(oracle):
    """The target is what the path itself produces from 6 of 40 atoms with known scales;
    the selection must find exactly them, and assembling with what it returns must
    reproduce the target."""
    wl = sr_synth.Workload("plant", 31, 2, 3, 20, 26, 4, 40, 5, "f16", "f32", 0.0, 1.0)
    inp = sr_synth.make_inputs(wl, DEV)
    planted = np.array([4, 9, 17, 22, 30, 39], dtype=np.int32)
    scales = np.array([1.5, 0.5, -1.0, 2.0, 0.75, 1.25], dtype=np.float32)
    target = torch.empty((wl.n, wl.c, wl.H, wl.W), device=DEV)
    sr.sr_dict_assemble_selective(inp["lr"], inp["coeff"], inp["dict"], wl.L, wl.k, wl.scale, wl.c, target,
                                  kept=planted, gamma=scales)
    up = torch.empty_like(target)
    sr.sr_bicubic_upsample(inp["lr"], wl.scale, wl.c, up)
    normal = sr.sr_atom_gram(up, inp["coeff"], inp["dict"], target, wl.L, wl.k, wl.c, stride=2)
    torch.cuda.synchronize()
    kept, gamma, lam = sr.sr_select_atoms(normal.cpu().numpy(), wl.L, alpha=6 / 40, delta_alpha=0.3)
    assert np.array_equal(kept, planted)
    assert np.allclose(gamma, scales, atol=2e-3)
    out = torch.empty_like(target)
    sr.sr_dict_assemble_selective(inp["lr"], inp["coeff"], inp["dict"], wl.L, wl.k, wl.scale, wl.c, out,
                                  kept=kept, gamma=gamma)
    torch.cuda.synchronize()
    assert float((out - target).abs().max()) <= 5e-3
    # the oracle's selection from the oracle's normal equations agrees
    U = oracle.bicubic(inp["lr"].cpu().numpy(), wl.scale)
    G0, b0, hh0, M0 = so.normal_equations(U, inp["coeff"].cpu().numpy(), inp["dict"].cpu().numpy(),
                                          target.cpu().numpy(), 2)
    k0, g0, _ = so.select_atoms(G0, b0, hh0, M0, 6 / 40, 0.3)
    assert np.array_equal(k0, kept) and np.allclose(g0, gamma, atol=2e-3)


def test_selection_finds_the_dominant_atoms_of_the_selective_workload():
    """The selective workload gives 8 seeded atoms most of the coefficient mass.  Asked for
    8 of 72 atoms to reproduce the DENSE result, Alg. 1 must pick exactly those 8 (the
    list the workload itself derives from the mean coefficients), and assembling with its
    kept list and gamma must come closer to the dense result than the unscaled kept list."""
    wl = sr_synth.scaled(sr_synth.WORKLOADS["4k_selective"], h=90, w=120)
    inp = sr_synth.make_inputs(wl, DEV)
    shape = (wl.n, wl.c, wl.H, wl.W)
    dense, up = torch.empty(shape, device=DEV), torch.empty(shape, device=DEV)
    sr.sr_dict_assemble(inp["lr"], inp["coeff"], inp["dict"], wl.L, wl.k, wl.scale, wl.c, dense)
    sr.sr_bicubic_upsample(inp["lr"], wl.scale, wl.c, up)
    normal = sr.sr_atom_gram(up, inp["coeff"], inp["dict"], dense, wl.L, wl.k, wl.c, stride=3)
    torch.cuda.synchronize()
    kept, gamma, _ = sr.sr_select_atoms(normal.cpu().numpy(), wl.L, alpha=8 / 72, delta_alpha=0.2)
    assert np.array_equal(kept, inp["kept"])
    assert np.array_equal(np.sort(sr_synth.dominant_atoms(wl)), kept)
    assert np.all(gamma > 1.0) and np.all(gamma < 1.5)          # they make up for the dropped ~13 % of the mass
    plain, scaled = torch.empty(shape, device=DEV), torch.empty(shape, device=DEV)
    sr.sr_dict_assemble_selective(inp["lr"], inp["coeff"], inp["dict"], wl.L, wl.k, wl.scale, wl.c, plain, kept=kept)
    sr.sr_dict_assemble_selective(inp["lr"], inp["coeff"], inp["dict"], wl.L, wl.k, wl.scale, wl.c, scaled,
                                  kept=kept, gamma=gamma)
    torch.cuda.synchronize()
    err_plain = float(((plain - dense) ** 2).mean())
    err_scaled = float(((scaled - dense) ** 2).mean())
    assert err_scaled < 0.25 * err_plain


def _reference(up, coeff, d, target, stride):
    """[L + 1][L + 1]: the products of the responses and the target, in 64 bits; and by atom the 2-norm, over the samples, of what bounds a
    response: coefficient x largest of the sample's taps x sum of the atom's magnitudes (for the target: its own)."""
    n, c, h, w = up.shape
    L, k = coeff.shape[1], d.shape[-1]
    r = (k - 1) // 2
    taps = torch.nn.functional.pad(up.double(), (r, r, r, r), mode="replicate")
    out = torch.zeros((L + 1, L + 1), device=DEV, dtype=torch.float64)
    most = torch.zeros(L, device=DEV, dtype=torch.float64)
    for b in range(n):
        phi = coeff[b].double()[:, ::stride, ::stride].reshape(L, -1)
        for ch in range(c):
            patch = torch.stack([taps[b, ch, i // k:i // k + h, i % k:i % k + w][::stride, ::stride].reshape(-1) for i in range(k * k)])
            resp = torch.cat([(d.reshape(L, -1).double() @ patch) * phi, target[b, ch].double()[::stride, ::stride].reshape(1, -1)])
            out += resp @ resp.T.contiguous()
            most += ((phi * patch.abs().amax(dim=0)) ** 2).sum(dim=1)
    most = torch.sqrt(most) * d.reshape(L, -1).double().abs().sum(dim=1)
    return out.cpu().numpy(), np.append(most.cpu().numpy(), np.sqrt(out[L, L].item()))


def _matrix(got, L):
    full = np.empty((L + 1, L + 1))
    full[:L, :L], full[L, :L], full[:L, L], full[L, L] = got[:L * L].reshape(L, L), got[L * L:L * L + L], got[L * L:L * L + L], got[L * L + L]
    return full


# Calls of 6144 items of 16 samples and one channel and more (several for a wavefront), fewer items for some wavefronts than for others: rows whose last item
# has 1, 4, 13 and 16 samples, every pixel and a lattice, several images, both block counts at an edge (the last block may hold the target only)
MANY = [(1, 3, 250, 417, 72, 5, "f16", 1), (2, 2, 213, 260, 79, 5, "f32", 1), (1, 1, 1100, 1197, 64, 5, "bf16", 1), (1, 3, 241, 353, 72, 5, "f8", 1),
         (1, 3, 500, 833, 72, 5, "f16", 2), (3, 1, 790, 1029, 63, 5, "f8", 3), (1, 4, 181, 417, 48, 5, "f32", 1), (1, 3, 250, 420, 47, 5, "f16", 1),
         (1, 3, 261, 433, 72, 3, "bf16", 1), (1, 3, 520, 865, 66, 3, "f32", 2), (1, 3, 270, 433, 60, 7, "f16", 1), (1, 2, 520, 1000, 31, 7, "f8", 2)]


@pytest.mark.parametrize("n,c,h,w,L,k,cd,stride", MANY)
@pytest.mark.parametrize("values", ["plain", "dark first", "peaks"])
def test_many_samples(n, c, h, w, L, k, cd, stride, values):
    """plain: coefficients as a softmax gives them.  dark first: no light in the upper rows, then 1e-6 of it, then all.
    peaks: single pixels of the image and coefficients far above the others."""
    g = torch.Generator(device=DEV).manual_seed(L * 1000 + w)
    up, target = (torch.rand((n, c, h, w), generator=g, device=DEV) for _ in range(2))
    z = torch.randn((n, L, h, w), generator=g, device=DEV)
    d = torch.randn((L, k, k), generator=g, device=DEV) / k
    if values == "dark first":
        up[:, :, :h // 3] = 0
        target[:, :, :h // 4] = 0
        up[:, :, h // 3:h // 2] *= 1e-6
    if values == "peaks":
        for t in (up, z, target):
            t.view(-1)[torch.randint(0, t.numel(), (40,), generator=g, device=DEV)] *= 300 if t is not z else 4
    phi = torch.softmax(z, dim=1)
    coeff = phi.to({"f32": torch.float32, "f16": torch.float16, "bf16": torch.bfloat16, "f8": torch.float8_e4m3fn}[cd])
    got = sr.sr_atom_gram(up, coeff, d, target, L, k, c, stride).cpu().numpy()
    again = sr.sr_atom_gram(up, coeff, d, target, L, k, c, stride).cpu().numpy()
    stored = coeff.float()
    ref, most = _reference(up, stored, d, target, stride)
    assert np.array_equal(got, again) and got[-1] == n * c * len(range(0, h, stride)) * len(range(0, w, stride))
    # the dot product of a response rounds to 2^-24 of its partial sums, each well below `most`, and the response to 2^-24 of itself: Cauchy-Schwarz over the
    # samples; sums round to 2^-24 of themselves, and over so many samples roundings average out
    size = np.sqrt(np.diag(ref))
    bound = 2.0 ** -24 * (np.outer(most + size, size) + np.outer(size, most + size) + np.outer(size, size))
    assert (np.abs(_matrix(got, L) - ref) <= bound).all()
    if values == "plain":
        # roundings of either sign: over 10^5 samples they average out (a cut towards zero, 2^-25 of a product, would be seen: 3e-8)
        assert np.abs(_matrix(got, L) - ref).sum() <= 1e-7 * np.abs(ref).sum()
        assert abs(((_matrix(got, L) - ref) / np.outer(size, size)).mean()) <= 4e-9


@pytest.mark.parametrize("where", ["coefficient inf", "coefficient nan", "image inf", "image nan", "dictionary inf", "target nan"])
def test_many_samples_with_infinities_and_nan(where):
    """They reach the sums they take part in, as fp32 products would, and no other; those stay as near as before."""
    n, c, h, w, L, k = 1, 3, 250, 420, 72, 5
    g = torch.Generator(device=DEV).manual_seed(11)
    up, target = (torch.rand((n, c, h, w), generator=g, device=DEV) for _ in range(2))
    coeff = torch.softmax(torch.randn((n, L, h, w), generator=g, device=DEV), dim=1)
    d = torch.rand((L, k, k), generator=g, device=DEV) + 0.1                   # (all positive: an infinity stays one)
    what, value = where.split()
    {"coefficient": coeff[0, 70], "image": up[0, 1], "dictionary": d[70], "target": target[0, 2]}[what].view(-1)[
        {"coefficient": 210 * w + 5, "image": 200 * w + 7, "dictionary": 3, "target": 99 * w + 33}[what]] = float(value)
    got = _matrix(sr.sr_atom_gram(up, coeff, d, target, L, k, c, 1).cpu().numpy(), L)
    hit = np.zeros(L + 1, bool)
    hit[{"coefficient": [70], "image": range(L), "dictionary": [70], "target": [L]}[what]] = True
    mine = hit[:, None] | hit[None, :]
    assert not np.isfinite(got[mine]).any() and (value != "inf" or np.isposinf(got[mine]).all())
    for t in (coeff, up, d, target):
        t.nan_to_num_(0.0, 0.0, 0.0)
    ref, _ = _reference(up, coeff, d, target, 1)
    size = np.sqrt(np.diag(ref))
    if what != "image":                              # (positive values: a response is as large as what bounds it, within a few times)
        assert (np.abs(got - ref) <= 1e-6 * np.outer(size, size))[~mine].all()


def _fp32_bound(up, coeff, d, target, stride):
    """Of each entry, for responses and sums formed in fp32: k^2 roundings of the dot product and one of the response, for both factors, and
    64 of the sum, each of 2^-24 of what the magnitudes add up to."""
    size, _ = _reference(up.abs(), coeff.abs(), d.abs(), target.abs(), stride)
    return (2 * (d.shape[-1] ** 2 + 1) + 64) * 2.0 ** -24 * size


@pytest.mark.parametrize("n,c,h,w,L,k,cd,stride", MANY)
@pytest.mark.parametrize("values", ["atoms", "coefficients", "outlier"])
def test_many_samples_of_atoms_of_any_magnitude(n, c, h, w, L, k, cd, stride, values):
    """Each entry as near as fp32 has it, however small its atoms' responses are beside the others': atoms (or their coefficients) of 2^-20 to
    2^-40 of the largest, or one response far above all others."""
    g = torch.Generator(device=DEV).manual_seed(L * 1000 + w)
    up, target = (torch.rand((n, c, h, w), generator=g, device=DEV) for _ in range(2))
    phi = torch.softmax(torch.randn((n, L, h, w), generator=g, device=DEV), dim=1)
    d = torch.randn((L, k, k), generator=g, device=DEV) / k
    small = torch.ones(L, device=DEV)
    if values == "outlier":
        phi[0, L // 2, 0, 0] = 400.0
        d[L // 2] *= 2.0 ** 30
    else:
        small[1::2] = 2.0 ** -torch.linspace(20, 40, L, device=DEV)[1::2].round()
    if values == "coefficients" and cd in ("f32", "bf16"):
        phi *= small[None, :, None, None]
    else:                                            # (fp16 and 8 bits do not hold such coefficients)
        d *= small[:, None, None]
    coeff = phi.to({"f32": torch.float32, "f16": torch.float16, "bf16": torch.bfloat16, "f8": torch.float8_e4m3fn}[cd])
    got = _matrix(sr.sr_atom_gram(up, coeff, d, target, L, k, c, stride).cpu().numpy(), L)
    ref, _ = _reference(up, coeff.float(), d, target, stride)
    assert (np.abs(got - ref) <= _fp32_bound(up, coeff.float(), d, target, stride)).all()


@pytest.mark.parametrize("sharp", [1, 10, 30])
@pytest.mark.parametrize("c,L,k,cd,stride", [(3, 72, 5, "f32", 1), (3, 72, 5, "f16", 1), (1, 72, 3, "bf16", 1), (3, 60, 7, "f32", 1), (3, 72, 5, "f32", 2)])
def test_many_samples_of_sharp_coefficients(c, L, k, cd, stride, sharp):
    """Softmax of Gaussian logits times `sharp`: few samples make up an entry then, and within the samples that an atom dominates the others' coefficients are tiny."""
    g = torch.Generator(device=DEV).manual_seed(sharp * 100 + L)
    h, w = (500, 833) if stride == 2 else (330, 833)
    up, target = (torch.rand((1, c, h, w), generator=g, device=DEV) for _ in range(2))
    phi = torch.softmax(sharp * torch.randn((1, L, h, w), generator=g, device=DEV), dim=1)
    d = torch.rand((L, k, k), generator=g, device=DEV) / k
    coeff = phi.to({"f32": torch.float32, "f16": torch.float16, "bf16": torch.bfloat16}[cd])
    got = _matrix(sr.sr_atom_gram(up, coeff, d, target, L, k, c, stride).cpu().numpy(), L)
    ref, _ = _reference(up, coeff.float(), d, target, stride)
    off = np.abs(got - ref) / ref                    # (all values are positive)
    # an entry of one sample is off by the roundings of two dot products, k^2 of either sign and up to 2^-25 of a partial sum each: their rms is k / 4 x 2^-24, and
    # less where several samples make up the entry (fp32 sums: largest 3.0e-8 to 7.4e-8, median up to 1.4e-8)
    assert off.max() <= 2.0 ** -23 and np.median(off) <= 2.0 ** -25


@pytest.mark.parametrize("n,c,h,w,L,k,cd,stride", MANY)
@pytest.mark.parametrize("what", ["image", "target", "coefficient"])
def test_many_samples_that_start_tiny(n, c, h, w, L, k, cd, stride, what):
    """Finite values of any magnitude give finite sums: a dictionary of 1e-5 and rows of 1e-30 before ordinary ones; a target, or coefficients, that go from
    1e-30 to 1e9."""
    if what == "coefficient" and cd not in ("f32", "bf16"):
        pytest.skip("the type holds no such coefficients")
    g = torch.Generator(device=DEV).manual_seed(L * 1000 + w)
    up, target = (torch.rand((n, c, h, w), generator=g, device=DEV) for _ in range(2))
    phi = torch.softmax(torch.randn((n, L, h, w), generator=g, device=DEV), dim=1)
    d = torch.randn((L, k, k), generator=g, device=DEV) / k
    row = torch.arange(h, device=DEV) % 8            # (wavefronts own runs of rows: each meets the change)
    ramp = torch.where(row < 4, 1e-30, 1e9 if what != "image" else 1.0).reshape(-1, 1) * torch.ones(w, device=DEV)
    if what == "image":
        up *= ramp
        d *= 1e-5
    elif what == "target":
        target *= ramp
    else:
        phi *= ramp
    coeff = phi.to({"f32": torch.float32, "f16": torch.float16, "bf16": torch.bfloat16, "f8": torch.float8_e4m3fn}[cd])
    got = _matrix(sr.sr_atom_gram(up, coeff, d, target, L, k, c, stride).cpu().numpy(), L)
    ref, _ = _reference(up, coeff.float(), d, target, stride)
    assert np.isfinite(got).all() and (np.abs(got - ref) <= _fp32_bound(up, coeff.float(), d, target, stride)).all()
