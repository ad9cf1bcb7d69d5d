"""The kernels at the sizes where their tiles, windows and size rules end, against the oracle.

Scores follow the tolerance of parity_util; selection and allocation are bit-exact; decode attention
follows |err| <= 5e-5 max|V| (fp32 exp2 and sums over up to N rows).
"""
import numpy as np
import pytest

import kvsynth
from oracle import flashcache_ref as ref

import parity_util as pu

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def _smooth_plus_noise(rng, shape, dtype):
    """[..., N, d]: a few low cosine modes, noise a tenth as strong, strongly deviating tokens."""
    n, d = shape[-2:]
    u = (np.arange(n) + 0.5) / n
    modes = np.cos(np.pi * u[:, None] * np.arange(6))
    x = modes @ rng.standard_normal(shape[:-2] + (6, d)) + 0.1 * rng.standard_normal(shape)
    x[..., rng.choice(n, max(1, n // 50), replace=False), :] += 3.0 * rng.standard_normal(d)
    x = x.astype(np.float32)
    return kvsynth.f32_to_bf16_bits(x) if dtype == "bf16" else x


# (tokens, kept modes, head_dim, dtype, heads).  The grid is the shortest of 2^k and 3 * 2^k points, from 64 to
# 16384, with 1.75 r points and N/16 points: every length once, at cut-offs that just fit it or are just above the
# shorter one, token counts one off a multiple of the 16-token tiles and 32-token steps, the fewest (256) and most
# tokens per grid point (16), and 1, 2 and 4 waves per unit (head_dim up to 64, 128, 256)
GRIDS = [(256, 1, 64, "f32", 2), (1024, 36, 8, "bf16", 3), (999, 54, 128, "bf16", 2), (2048, 73, 72, "f32", 1),
         (1025, 109, 136, "bf16", 2), (257, 128, 128, "bf16", 5), (513, 146, 256, "bf16", 1), (777, 219, 64, "bf16", 2),
         (1111, 292, 128, "f32", 1), (1533, 438, 40, "bf16", 2), (2047, 585, 128, "bf16", 9), (3001, 877, 128, "bf16", 2),
         (3333, 1170, 16, "f32", 2), (4099, 1755, 64, "bf16", 1), (9001, 2340, 24, "bf16", 2), (7023, 3510, 8, "bf16", 2),
         (9401, 4680, 16, "f32", 1), (14055, 7022, 8, "bf16", 1), (18749, 9362, 16, "bf16", 1),
         (100003, 100, 8, "bf16", 1), (262144, 40, 8, "bf16", 1)]


@pytest.mark.parametrize("n,r,d,dtype,heads", GRIDS)
def test_scores_at_every_grid_length(n, r, d, dtype, heads):
    import paper_2511_16786_amd as fc
    rng = np.random.default_rng(n + r)
    K = _smooth_plus_noise(rng, (1, 1, heads, n, d), dtype)
    V = _smooth_plus_noise(rng, (1, 1, heads, n, d), dtype)
    want = ref.score(K, V, dtype, r, route="fast")
    Kt, Vt = pu.to_torch(K, dtype), pu.to_torch(V, dtype)
    comp = fc.Compressor(Kt, r, ref.total_budget(1, n, 0.2))
    comp.run(Kt, Vt)
    torch.cuda.synchronize()
    assert fc.workspace_error(comp.workspace) == 0
    pu.check_scores(comp.scores.cpu().numpy(), want["score"], pu.unit_power(ref.widen(K, dtype), ref.widen(V, dtype)))
    e = comp.energy.cpu().numpy()
    assert np.allclose(e[..., 2:], want["energy"][..., 2:], rtol=1e-5)
    assert np.all(np.abs(e[..., :2] - want["energy"][..., :2]) <= 1e-4 * want["energy"][..., :2]
                  + 1e-7 * want["energy"][..., 2:])


# One wave of the residual kernel holds columns of both tensors (64: all of them, 72 and 136: across the seam; 128: none)
@pytest.mark.parametrize("d", [64, 72, 128, 136])
@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_energies_of_tensors_many_octaves_apart(d, dtype):
    """K and V are scored by themselves: each energy keeps its accuracy however small its tensor is beside the other
    (multiplied by powers of two, which round nothing)."""
    import paper_2511_16786_amd as fc
    rng = np.random.default_rng(d)
    n, r = 1024, 52
    X = _smooth_plus_noise(rng, (2, 1, 1, 1, n, d), "f32")
    if dtype == "bf16":
        X = ref.widen(kvsynth.f32_to_bf16_bits(X), "bf16").astype(np.float32)

    def stored(x):
        return kvsynth.f32_to_bf16_bits(x) if dtype == "bf16" else x
    for k in (12, 24, 30, 34, 40, 50):
        for small in (0, 1):
            K, V = (stored(x * np.float32(2.0 ** -k if t == small else 1.0)) for t, x in enumerate(X))
            want = ref.score(K, V, dtype, r, route="fast")["energy"]
            Kt, Vt = pu.to_torch(K, dtype), pu.to_torch(V, dtype)
            comp = fc.Compressor(Kt, r, ref.total_budget(1, n, 0.2))
            comp.run_score(Kt, Vt)
            e = comp.energy.cpu().numpy()
            assert np.all(np.abs(e[..., :2] - want[..., :2]) <= 1e-4 * want[..., :2] + 1e-7 * want[..., 2:]), (k, small)
            assert np.allclose(e[..., 2:], want[..., 2:], rtol=1e-5), (k, small)


def _residual64(X, r):
    """K or V [.., N, d] on the GPU without its r lowest modes, in 64 bits from the basis itself."""
    n, d = X.shape[-2:]
    x = X.double().reshape(-1, n, d)
    i = torch.arange(n, device="cuda", dtype=torch.float64) + 0.5
    base = torch.zeros_like(x)
    for a in range(0, r, 1024):
        m = torch.arange(a, min(r, a + 1024), device="cuda", dtype=torch.float64)
        basis = torch.cos(np.pi / n * m[:, None] * i) * np.sqrt(2.0 / n)
        if a == 0:
            basis[0] *= np.sqrt(0.5)
        for u in range(x.shape[0]):
            base[u] += basis.t().contiguous() @ (basis @ x[u])
    return (x - base).reshape(X.shape)


# 1, 2 and 4 waves per unit, with waves that take the parts of a unit in turn and side by side
@pytest.mark.parametrize("n,r,d,units", [(1000, 50, 64, 8), (4096, 205, 128, 8), (4096, 64, 256, 8), (512, 20, 128, 900)])
@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_sums_of_noise_are_as_good_as_64_bits(n, r, d, units, dtype):
    """White columns leave the sums themselves as the error.  Energies: up to 32 squares are added in fp32 and the rest
    in fp64, at most 32 * 2^-24 and by chance 1e-7 / sqrt(n d / 32) < 1e-8; scores: one rounding to fp32, 2.5e-8 in
    the mean, beside sums over 8 columns and 4 lanes of 1.9e-8 (d = 64: 4 of its 8 slots at once, 2.7e-8)."""
    import paper_2511_16786_amd as fc
    gen = torch.Generator(device="cuda")
    gen.manual_seed(n + d)
    K, V = (torch.randn((1, 1, units, n, d), generator=gen, device="cuda").to(
        torch.bfloat16 if dtype == "bf16" else torch.float32) for _ in range(2))
    comp = fc.Compressor(K, r, ref.total_budget(1, n, 0.2))
    comp.run_score(K, V)
    hp = [_residual64(X, r) for X in (K, V)]
    want = torch.stack([x.pow(2).sum((-1, -2)) for x in (hp[0], hp[1], K.double(), V.double())], -1)
    off = (comp.energy / want - 1.0).abs().amax((0, 1, 2)).tolist()
    assert max(off[:2]) <= 4e-9
    # (bf16 squares have 16 bits, and 8 of them added in fp32, rounded to nearest, come out 6.5e-9 low in the mean)
    assert max(off[2:]) <= (1e-8 if dtype == "bf16" else 4e-9)
    s = (hp[0].pow(2).sum(-1) + hp[1].pow(2).sum(-1)) / d
    assert float((comp.scores.double() - s).norm() / s.norm()) <= (4.0e-8 if d == 64 else 3.6e-8)


# Every grid length from 128 points on at cut-offs near N/4, from where on grids of up to 4096 points are transformed in
# 64 bits, and near N/2
@pytest.mark.parametrize("n,r", [(260, 64), (260, 66), (300, 76), (420, 106), (600, 151), (777, 219), (512, 231),
                                 (1111, 293), (2048, 512), (2048, 513), (3072, 877), (3001, 991), (4099, 1755),
                                 (7680, 2305), (4000, 990), (7023, 3400), (9401, 4680), (12544, 5645), (18749, 9362)])
@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_scores_at_high_cutoffs_are_as_good_as_64_bits(n, r, dtype):
    """What remains above a high cut-off is small beside the columns, and their transform's rounding counts.  Allowed
    are four times the 2.5e-8 of one rounding to fp32 (of the score, its sums, the weights and the grid values), and
    1.7e-7 for grids of more than 4096 points, whose transform adds sqrt(2 log2 M) roundings of 2.5e-8, 1.3e-7."""
    import paper_2511_16786_amd as fc
    rng = np.random.default_rng(n + r)
    K, V = (pu.to_torch(_smooth_plus_noise(rng, (1, 1, 2, n, 64), dtype), dtype) for _ in range(2))
    comp = fc.Compressor(K, r, ref.total_budget(1, n, 0.2))
    comp.run_score(K, V)
    hp = [_residual64(X, r) for X in (K, V)]
    s = (hp[0].pow(2).sum(-1) + hp[1].pow(2).sum(-1)) / 64
    assert float((comp.scores.double() - s).norm() / s.norm()) <= (1e-7 if 7 * r <= 4 * 4096 else 1.7e-7)


@pytest.mark.parametrize("n,r", [(1024, 292), (2048, 585), (3072, 877), (7680, 2305)])
def test_modes_just_below_the_cutoff_are_kept(n, r):
    """Few grid points per mode (1.75): the last kept mode is what the window and the rounding of the grid's points,
    which comes back 1 / phihat(r) = 6.6 times as large, reproduce worst: window 4.6e-8, points 6.6 * 2.5e-8, the rest
    of the way 1e-7, together 2e-7 of the mode, by chance a third more."""
    import paper_2511_16786_amd as fc
    lost = []
    for m in (r - 1, r - 2):
        x = np.cos(np.pi * m * (np.arange(n) + 0.5) / n)
        for scale in (1.0, 1.17, 1.34, 1.51):
            X = torch.from_numpy(np.repeat(scale * x[:, None], 8, 1).astype(np.float32)[None, None, None]).cuda()
            comp = fc.Compressor(X, r, ref.total_budget(1, n, 0.2))
            comp.run_score(X, X)
            e = comp.energy[0, 0, 0]
            lost.append(float(e[0] / e[2]))
    assert np.sqrt(np.mean(lost)) <= 2.7e-7


# What the resampled transform leaves to the other two: 9363 modes to where the grid of 24576 points is taken, above N/2, above head_dim 256
@pytest.mark.parametrize("path,n,r,d", [("basis", 20011, 9363, 16), ("basis", 20011, 9900, 64), ("basis", 20011, 10100, 64),
                                        ("stream", 20480, 9363, 16), ("stream", 20480, 9900, 64),
                                        ("stream", 20480, 10241, 8), ("stream", 2048, 200, 264), ("stream", 2560, 600, 272)])
@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_shapes_left_to_the_basis_and_the_streaming_transform(path, n, r, d, dtype):
    import paper_2511_16786_amd as fc
    rng = np.random.default_rng(n + r)
    K = _smooth_plus_noise(rng, (1, 1, 2, n, d), dtype)
    V = _smooth_plus_noise(rng, (1, 1, 2, n, d), dtype)
    Kt, Vt = pu.to_torch(K, dtype), pu.to_torch(V, dtype)
    comp = fc.Compressor(Kt, r, ref.total_budget(1, n, 0.2))
    assert fc.realisation(comp.desc, r) == fc.binding.PATHS[path]
    comp.run(Kt, Vt)
    assert fc.workspace_error(comp.workspace) == 0
    want = ref.score(K, V, dtype, r, route="fast")
    pu.check_scores(comp.scores.cpu().numpy(), want["score"], pu.unit_power(ref.widen(K, dtype), ref.widen(V, dtype)))
    e = comp.energy.cpu().numpy()
    assert np.allclose(e[..., 2:], want["energy"][..., 2:], rtol=1e-5)
    assert np.all(np.abs(e[..., :2] - want["energy"][..., :2]) <= 1e-4 * want["energy"][..., :2]
                  + 1e-7 * want["energy"][..., 2:])


@pytest.mark.parametrize("layout", ["token_major", "padded_rows", "heads_last"])
@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_scores_do_not_depend_on_strides(layout, dtype):
    """The same values behind other strides give the same bits (odd token count, batch and layers)."""
    import paper_2511_16786_amd as fc
    rng = np.random.default_rng(5)
    B, L, H, n, d = 2, 2, 3, 1237, 64
    dense = [pu.to_torch(_smooth_plus_noise(rng, (B, L, H, n, d), dtype), dtype) for _ in range(2)]

    def lay(x):
        if layout == "token_major":
            return x.permute(0, 1, 3, 2, 4).contiguous().permute(0, 1, 3, 2, 4)
        if layout == "padded_rows":
            wide = torch.zeros((B, L, H, n + 3, d + 8), dtype=x.dtype, device=x.device)
            wide[:, :, :, :n, :d] = x
            return wide[:, :, :, :n, :d]
        return x.permute(2, 1, 0, 3, 4).contiguous().permute(2, 1, 0, 3, 4)
    got = []
    for K, V in (dense, [lay(x) for x in dense]):
        comp = fc.Compressor(K, 124, ref.total_budget(L, n, 0.2))
        comp.run(K, V)
        torch.cuda.synchronize()
        got.append((comp.scores.cpu(), comp.energy.cpu(), comp.idx.cpu()))
    for a, b in zip(*got):
        assert torch.equal(a, b)


@pytest.mark.parametrize("bad", [float("inf"), float("nan")])
def test_a_value_that_is_not_finite_spoils_its_own_unit_only(bad):
    """Base KV of a column that holds it is not finite anywhere; other units' scores keep their bits."""
    import paper_2511_16786_amd as fc
    rng = np.random.default_rng(8)
    n = 1500
    K, V = (pu.to_torch(_smooth_plus_noise(rng, (1, 2, 4, n, 64), "bf16"), "bf16") for _ in range(2))
    comp = fc.Compressor(K, 150, ref.total_budget(2, n, 0.2))
    comp.run_score(K, V)
    clean = comp.scores.clone()
    K[0, 1, 2, 700, 5] = bad
    comp.run_score(K, V)
    torch.cuda.synchronize()
    same = torch.ones((2, 4), dtype=torch.bool)
    same[1, 2] = False
    for l in range(2):
        for h in range(4):
            if same[l, h]:
                assert torch.equal(comp.scores[0, l, h], clean[0, l, h])
            else:
                assert not torch.isfinite(comp.scores[0, l, h]).any()


# one key, and both sides of every size at which the selection kernel changes
@pytest.mark.parametrize("n", [1, 63, 1024, 1025, 4096, 4097, 8192, 8193, 16385, 32768, 32769, 65536, 65537])
@pytest.mark.parametrize("shared", [False, True])
def test_selection_of_uneven_key_ranges(n, shared):
    """Scores that fill the search's bins unevenly: equal ones, two values, one far above the others, many
    magnitudes, both signs, infinities, and a NaN of all set bits beside others."""
    import paper_2511_16786_amd as fc
    rng = np.random.default_rng(n)
    L, d = 6, 8
    s = np.empty((1, L, 1, n), np.float32)
    s[0, 0] = 0.5
    s[0, 1] = np.where(rng.uniform(size=n) < 0.3, np.float32(1.0), np.nextafter(np.float32(1.0), np.float32(2.0)))
    s[0, 2] = rng.uniform(0.01, 0.02, n)
    s[0, 2, 0, n // 2] = 3e38
    s[0, 3] = np.exp(rng.uniform(-80, 80, n))
    s[0, 4] = rng.standard_normal(n)
    s[0, 4, 0, n // 3] = np.inf
    s[0, 5] = rng.gamma(2.0, 1.0, n)
    s[0, 5, 0, n // 4] = np.array(0xFFFFFFFF, np.uint32).view(np.float32)
    K = rng.standard_normal((1, L, 1, n, d)).astype(np.float32)
    Kt = torch.from_numpy(K).cuda()
    s_t = torch.from_numpy(s).cuda()
    bits = s.view(np.uint32)
    key = np.where(bits >> 31, ~bits, bits | np.uint32(1 << 31))
    if shared:                           # (the head mean's division may give the NaN another payload)
        key[np.isnan(s)] = 0
    for k in sorted({1, (n + 1) // 2, max(1, n - 1), n}):
        budgets = np.full((1, L), k, np.int64)
        offs = ref.layer_offsets(budgets[0], 1)
        rows = int(offs[-1])
        idx = torch.full((1, rows), -1, dtype=torch.int32, device="cuda")
        Ko = torch.zeros((1, rows, d), device="cuda")
        Vo = torch.zeros_like(Ko)
        fc.select_gather(Kt, Kt, fc.describe(Kt), s_t, torch.from_numpy(budgets.astype(np.int32)).cuda(),
                         torch.from_numpy(offs[None]).cuda(), rows, idx, Ko, Vo, shared=shared)
        got = idx.cpu().numpy()[0]
        for l in range(5 if shared else L):
            order = np.lexsort((np.arange(n), -key[0, l, 0].astype(np.int64)))
            assert np.array_equal(got[l * k:(l + 1) * k], np.sort(order[:k])), (l, k)


# every remainder of the four scores a lane loads, units that begin at any multiple of 4 bytes, ties within and across waves;
# rows of 1, 3, 9, 32 and 257 vectors of 16 bytes, fewer kept rows than a workgroup takes, and many layers
@pytest.mark.parametrize("n,L,H,d,dtype", [(1, 70, 1, 8, "bf16"), (2, 70, 3, 24, "bf16"), (3, 9, 2, 72, "bf16"), (5, 3, 3, 128, "f32"),
                                           (6, 2, 1, 2056, "bf16"), (1021, 70, 3, 8, "bf16"), (2046, 3, 2, 72, "bf16"),
                                           (4095, 2, 3, 128, "f32"), (16381, 2, 3, 24, "bf16"), (40002, 2, 1, 8, "bf16")])
@pytest.mark.parametrize("shared", [False, True])
def test_selection_and_gather_of_odd_sizes(n, L, H, d, dtype, shared):
    import paper_2511_16786_amd as fc
    rng = np.random.default_rng(n + L)
    K, V = (rng.integers(0, 0x7F80, (L, H, n, d)).astype(np.uint16) if dtype == "bf16" else
            rng.standard_normal((L, H, n, d)).astype(np.float32) for _ in range(2))
    scores = rng.integers(0, 3 + n // 4, (L, H, n)).astype(np.float32)
    scores[::2] += rng.uniform(0.0, 0.5, (len(scores[::2]), H, n)).astype(np.float32)
    budgets = rng.integers(1, n + 1, L)
    budgets[0] = n
    want = ref.select_gather(K, V, scores, budgets, shared=shared)
    offs = ref.layer_offsets(budgets, H)
    rows = int(offs[-1])
    Kt, Vt = pu.to_torch(K[None], dtype), pu.to_torch(V[None], dtype)
    s_t, b_t, o_t = (torch.from_numpy(x[None]).cuda() for x in (scores, budgets.astype(np.int32), offs))
    idx = torch.full((1, rows), -1, dtype=torch.int32, device="cuda")
    Ko, Vo = (torch.zeros((1, rows, d), dtype=Kt.dtype, device="cuda") for _ in range(2))
    fc.select_gather(Kt, Vt, fc.describe(Kt), s_t, b_t, o_t, rows, idx, Ko, Vo, shared=shared)
    assert np.array_equal(idx.cpu().numpy()[0], want["idx"])
    assert np.array_equal(pu.rows_to_numpy(Ko, dtype)[0], want["K_out"])
    assert np.array_equal(pu.rows_to_numpy(Vo, dtype)[0], want["V_out"])
    page = 3
    reach = -(-n // page)
    table = rng.permutation(L * H * reach).astype(np.int32).reshape(L, H, reach)
    Kc, Vc = (torch.zeros((L * H * reach, page, d), dtype=Kt.dtype, device="cuda") for _ in range(2))
    fc.select_gather_paged(Kt, Vt, fc.describe(Kt), s_t, b_t, o_t, rows, idx, torch.from_numpy(table[None]).cuda(), page, Kc, Vc,
                           shared=shared)
    for got, packed in ((Kc, want["K_out"]), (Vc, want["V_out"])):
        paged = np.zeros(got.shape, dtype=K.dtype)
        ref.scatter_paged(packed, budgets, H, table, page, paged)
        assert np.array_equal(pu.rows_to_numpy(got, dtype), paged)


@pytest.mark.parametrize("L", [63, 64, 65])
def test_allocation_on_both_sides_of_one_wave(L):
    import paper_2511_16786_amd as fc
    rng = np.random.default_rng(L)
    B, H, N = 40, 2, 300
    energy = np.empty((B, L, H, 4))
    energy[..., 2:] = rng.uniform(1.0, 100.0, (B, L, H, 2))
    energy[..., :2] = energy[..., 2:] * rng.uniform(0.0, 1.0, (B, L, H, 2)) ** 4
    energy[:, ::7, :, :2] = 0.0
    e_t = torch.from_numpy(energy).cuda()
    for T, lo, hi in ((L * 60, 1, N), (L * 60, 20, 90), (L * 90 - 1, 5, 90), (L, 1, N)):
        budgets = torch.empty((B, L), dtype=torch.int32, device="cuda")
        offs = torch.empty((B, L + 1), dtype=torch.int64, device="cuda")
        fc.allocate(e_t, B, L, H, N, T, lo, hi, budgets, offs)
        bg, og = budgets.cpu().numpy(), offs.cpu().numpy()
        for b in range(B):
            want, _ = ref.allocate(ref.layer_ratios(energy[b]), T, lo, hi)
            assert np.array_equal(bg[b], want)
            assert np.array_equal(og[b], ref.layer_offsets(want, H))


# budgets on both sides of a step (32 rows a wave) and of a 128-row piece; page sizes that do and do not divide a step
@pytest.mark.parametrize("page", [0, 1, 7, 16, 64, 200])
@pytest.mark.parametrize("dtype,d,group", [("bf16", 128, 7), ("bf16", 64, 16), ("f32", 128, 4)])
def test_decode_rows_that_end_inside_a_step(dtype, d, group, page):
    import paper_2511_16786_amd as fc
    rng = np.random.default_rng(17 * group + page)
    B, L, H = 1, 8, 2
    budgets = np.array([[1, 31, 32, 33, 127, 129, 640, 2049]], dtype=np.int64)
    offs = ref.layer_offsets(budgets[0], H)
    rows = int(offs[-1])

    def make(shape, sigma=1.0):
        x = (sigma * rng.standard_normal(shape)).astype(np.float32)
        return kvsynth.f32_to_bf16_bits(x) if dtype == "bf16" else x
    Kr, Vr, Q = make((B, rows, d)), make((B, rows, d), 2.0), make((B, L, H * group, d))
    scale = float(1.0 / np.sqrt(d))
    b_t = torch.from_numpy(budgets.astype(np.int32)).cuda()
    want = ref.decode_attention(Q[0], Kr[0], Vr[0], dtype, budgets[0], H, scale)
    if page == 0:
        out = fc.decode_attention(pu.to_torch(Q, dtype), pu.to_torch(Kr, dtype), pu.to_torch(Vr, dtype), H, b_t,
                                  torch.from_numpy(offs[None]).cuda(), rows, scale)
    else:
        reach = -(-int(budgets.max()) // page)
        pages = B * L * H * reach
        table = rng.permutation(pages).astype(np.int32).reshape(B, L, H, reach)
        Kc = np.zeros((pages, page, d), dtype=Kr.dtype)
        Vc = np.zeros_like(Kc)
        ref.scatter_paged(Kr[0], budgets[0], H, table[0], page, Kc)
        ref.scatter_paged(Vr[0], budgets[0], H, table[0], page, Vc)
        out = fc.decode_attention_paged(pu.to_torch(Q, dtype), pu.to_torch(Kc, dtype), pu.to_torch(Vc, dtype), H, b_t,
                                        torch.from_numpy(table).cuda(), scale)
    err = np.abs(out.cpu().numpy()[0] - want).max()
    assert err <= 5e-5 * float(np.abs(ref.widen(Vr, dtype)).max())


# launches whose workgroups take the layers by falling budget (2 to 64 of them), and one layer too many for that: layers
# with the same budget, with one row and with none, and sequences whose orders differ
@pytest.mark.parametrize("B,L,H", [(8, 2, 16), (2, 64, 2), (2, 65, 2)])
@pytest.mark.parametrize("dtype,group,page", [("bf16", 4, 0), ("bf16", 16, 16), ("f32", 2, 0), ("f32", 1, 48)])
def test_decode_of_many_long_pieces(B, L, H, dtype, group, page):
    import paper_2511_16786_amd as fc
    rng = np.random.default_rng(L + group)
    d, mean = 64, 1100
    budgets = np.empty((B, L), np.int64)
    for b in range(B):
        half = rng.integers(0, 2 * mean, L // 2)
        budgets[b] = rng.permutation(np.concatenate([half, 2 * mean - half, np.full(L % 2, mean)]))
    if L > 2:
        budgets[0, :6] = 1, 0, 1700, 1700, 2 * mean, 3 * mean - 1
    rows = max(H * mean * L, int(H * budgets.sum(axis=1).max()))
    offs = np.stack([ref.layer_offsets(k, H) for k in budgets])

    def make(shape, sigma=1.0):
        x = (sigma * rng.standard_normal(shape, dtype=np.float32)).astype(np.float32)
        return kvsynth.f32_to_bf16_bits(x) if dtype == "bf16" else x
    K, V, Q = make((B, rows, d)), make((B, rows, d), 2.0), make((B, L, H * group, d))
    scale = float(1.0 / np.sqrt(d))
    b_t = torch.from_numpy(budgets.astype(np.int32)).cuda()
    if page == 0:
        out = fc.decode_attention(pu.to_torch(Q, dtype), pu.to_torch(K, dtype), pu.to_torch(V, dtype), H, b_t,
                                  torch.from_numpy(offs).cuda(), rows, scale)
    else:
        reach = -(-int(budgets.max()) // page)
        table = rng.permutation(B * L * H * reach).astype(np.int32).reshape(B, L, H, reach)
        Kc = np.zeros((B * L * H * reach, page, d), dtype=K.dtype)
        Vc = np.zeros_like(Kc)
        for b in range(B):
            ref.scatter_paged(K[b], budgets[b], H, table[b], page, Kc)
            ref.scatter_paged(V[b], budgets[b], H, table[b], page, Vc)
        out = fc.decode_attention_paged(pu.to_torch(Q, dtype), pu.to_torch(Kc, dtype), pu.to_torch(Vc, dtype), H, b_t,
                                        torch.from_numpy(table).cuda(), scale)
    out = out.cpu().numpy()
    for b in range(B):
        want = ref.decode_attention(Q[b], K[b], V[b], dtype, budgets[b], H, scale)
        assert np.abs(out[b] - want).max() <= 5e-5 * float(np.abs(ref.widen(V[b], dtype)).max()), b


# sequences of one launch with long pieces, whose layers come by falling budget, and with short ones, whose layers do not; a table
# that reaches further than any budget
@pytest.mark.parametrize("dtype,d,group,page", [("bf16", 128, 4, 64), ("bf16", 64, 7, 16), ("f32", 64, 2, 0), ("bf16", 128, 2, 0), ("f32", 128, 1, 48)])
def test_decode_of_sequences_with_long_and_short_pieces(dtype, d, group, page):
    import paper_2511_16786_amd as fc
    rng = np.random.default_rng(d + group)
    B, L, H = 3, 44, 8                                           # (1056 units: one piece each)
    long = 88 * 1024 // (d * (2 if dtype == "bf16" else 4))      # rows of 88 KiB, on average
    budgets = np.stack([rng.permutation(np.linspace(lo, hi, L).astype(np.int64)) for lo, hi in ((0, 2 * long), (0, 180), (1, 1))])
    offs = np.stack([ref.layer_offsets(k, H) for k in budgets])
    rows = int(offs[0, -1])

    def make(shape, sigma=1.0):
        x = (sigma * rng.standard_normal(shape, dtype=np.float32)).astype(np.float32)
        return kvsynth.f32_to_bf16_bits(x) if dtype == "bf16" else x
    K, V, Q = make((B, rows, d)), make((B, rows, d), 2.0), make((B, L, H * group, d))
    scale = float(1.0 / np.sqrt(d))
    b_t = torch.from_numpy(budgets.astype(np.int32)).cuda()
    if page == 0:
        out = fc.decode_attention(pu.to_torch(Q, dtype), pu.to_torch(K, dtype), pu.to_torch(V, dtype), H, b_t,
                                  torch.from_numpy(offs).cuda(), rows, scale)
    else:
        reach = 8192 // page
        need = -(-budgets // page)
        table = np.full((B, L, H, reach), -1, np.int32)
        at = 0
        for b in range(B):
            for l in range(L):
                for h in range(H):
                    table[b, l, h, :need[b, l]] = np.arange(at, at + need[b, l])
                    at += int(need[b, l])
        Kc, Vc = np.zeros((at, page, d), dtype=K.dtype), np.zeros((at, page, d), dtype=K.dtype)
        for b in range(B):
            ref.scatter_paged(K[b], budgets[b], H, table[b], page, Kc)
            ref.scatter_paged(V[b], budgets[b], H, table[b], page, Vc)
        out = fc.decode_attention_paged(pu.to_torch(Q, dtype), pu.to_torch(Kc, dtype), pu.to_torch(Vc, dtype), H, b_t,
                                        torch.from_numpy(table).cuda(), scale)
    out = out.cpu().numpy()
    for b in range(B):
        want = ref.decode_attention(Q[b], K[b], V[b], dtype, budgets[b], H, scale)
        assert np.abs(out[b] - want).max() <= 5e-5 * float(np.abs(ref.widen(V[b], dtype)).max()), b


# few rows in buffers and pools of more than 256 MB, whose launches look at the budgets before they read past the last-level cache,
# and the same rows in small ones
@pytest.mark.parametrize("page", [0, 16])
@pytest.mark.parametrize("dtype,d,group", [("bf16", 128, 7), ("bf16", 64, 4), ("f32", 64, 2)])
def test_decode_of_large_caches_is_the_same_bits(dtype, d, group, page):
    import paper_2511_16786_amd as fc
    gen = torch.Generator(device="cuda").manual_seed(d + group)
    L, H = 4, 2
    budgets = [1, 200, 1025, 2047]
    offs = torch.tensor([[0] + [H * sum(budgets[:l + 1]) for l in range(L)]], device="cuda")
    rows = int(offs[0, -1])
    dt = torch.float32 if dtype == "f32" else torch.bfloat16
    Q = torch.randn((1, L, H * group, d), generator=gen, device="cuda").to(dt)
    b_t = torch.tensor([budgets], dtype=torch.int32, device="cuda")
    large = -(-(1 << 28) // (2 * d * Q.element_size()) // 16) * 16
    assert 2 * large * d * Q.element_size() >= 1 << 28 > 2 * 2 * rows * d * Q.element_size()
    K, V = (torch.randn((rows, d), generator=gen, device="cuda").to(dt) for _ in range(2))
    out = []
    for held in (-(-rows // 16) * 16 + 16 * L * H, large):
        Kc, Vc = (torch.zeros((held, d), dtype=dt, device="cuda") for _ in range(2))
        if page == 0:
            Kc[:rows], Vc[:rows] = K, V
            out.append(fc.decode_attention(Q, Kc[None], Vc[None], H, b_t, offs, held, 0.1))
            continue
        reach = max(160, held // (page * L * H))         # (both launches for more than 16 pieces: one order of the sums)
        table = (torch.arange(L * H * reach, dtype=torch.int32, device="cuda") % (held // page)).reshape(1, L, H, reach)
        first = 0
        for l in range(L):
            for h in range(H):
                need = -(-budgets[l] // page)
                table[0, l, h, :need] = torch.arange(first // page, first // page + need, dtype=torch.int32, device="cuda")
                at = int(offs[0, l]) + h * budgets[l]
                Kc[first:first + budgets[l]], Vc[first:first + budgets[l]] = K[at:at + budgets[l]], V[at:at + budgets[l]]
                first += need * page
        out.append(fc.decode_attention_paged(Q, Kc.view(-1, page, d), Vc.view(-1, page, d), H, b_t, table, 0.1))
    assert torch.equal(out[0], out[1])


# one sequence whose rows are read past the last-level cache, by what the launch reads if all are like it, and one whose rows are
# not, of one layer, of layers that may come by falling budget, and of more layers than a wave has lanes
@pytest.mark.parametrize("L,H", [(1, 8), (2, 8), (70, 2)])
@pytest.mark.parametrize("dtype,d,group,page", [("bf16", 128, 4, 0), ("bf16", 64, 7, 64), ("f32", 64, 2, 16), ("f32", 128, 8, 0)])
def test_decode_of_rows_past_the_cache_and_in_it(L, H, dtype, d, group, page):
    import paper_2511_16786_amd as fc
    gen = torch.Generator(device="cuda").manual_seed(L + d + group)
    B, scale = 2, 0.1
    dt = torch.float32 if dtype == "f32" else torch.bfloat16
    row_bytes = d * dt.itemsize
    many = -(-256_000_000 // (2 * row_bytes * B * L * H)) + 1
    budgets = torch.tensor([[many + 7 * (l % 3) for l in range(L)], [1 + 37 * l % 200 for l in range(L)]])
    assert 2 * row_bytes * B * H * int(budgets[0].sum()) > 256_000_000 > 2 * row_bytes * B * H * int(budgets[1].sum())
    offs = torch.zeros((B, L + 1), dtype=torch.int64)
    offs[:, 1:] = torch.cumsum(H * budgets, 1)
    rows = int(offs[:, -1].max())
    Q = torch.randn((B, L, H * group, d), generator=gen, device="cuda").to(dt)
    K, V = (torch.randn((B, rows, d), generator=gen, device="cuda").to(dt) for _ in range(2))
    b_t = budgets.to(torch.int32).cuda()
    if page == 0:
        out = fc.decode_attention(Q, K, V, H, b_t, offs.cuda(), rows, scale)
    else:
        need = -(-budgets // page)
        pages, reach = H * int(need.sum()), int(need.max()) + 3
        table = torch.full((B, L, H, reach), -1, dtype=torch.int32)
        Kc, Vc = (torch.zeros((pages, page, d), dtype=dt, device="cuda") for _ in range(2))
        at = 0
        for b in range(B):
            for l in range(L):
                for h in range(H):
                    k, first = int(budgets[b, l]), int(offs[b, l]) + h * int(budgets[b, l])
                    table[b, l, h, :need[b, l]] = torch.arange(at, at + int(need[b, l]), dtype=torch.int32)
                    for full, cache in ((K, Kc), (V, Vc)):
                        cache.view(-1, d)[at * page:at * page + k] = full[b, first:first + k]
                    at += int(need[b, l])
        out = fc.decode_attention_paged(Q, Kc, Vc, H, b_t, table.cuda(), scale)
    for b in range(B):
        for l in range(L):
            for h in range(H):
                k, first = int(budgets[b, l]), int(offs[b, l]) + h * int(budgets[b, l])
                q = Q[b, l, h * group:(h + 1) * group].double()
                p = torch.softmax(scale * (K[b, first:first + k].double() @ q.T), 0)
                want = p.T.contiguous() @ V[b, first:first + k].double()
                err = (out[b, l, h * group:(h + 1) * group].double() - want).abs().max()
                assert float(err) <= 5e-5 * float(V[b, first:first + k].abs().max()), (b, l, h)


# most layers keep less than the launch's pieces (units first), or more (a unit's pieces first)
@pytest.mark.parametrize("most", [57, 1300])
@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_decode_cuts_every_unit_by_its_own_budget(dtype, most):
    """Pieces of 128 rows and more, up to the launch's number for a unit, whatever the other layers keep: a record per
    piece is written, and no other.  The result is the same as for the unit by itself up to the order of the sums."""
    import paper_2511_16786_amd as fc
    rng = np.random.default_rng(3)
    L, H, group, d = 28, 4, 7, 128
    budgets = np.full(L, most, np.int64)
    budgets[[3, 11, 20, 27]] = 2048, 0, 129, 1000
    offs = ref.layer_offsets(budgets, H)
    rows = int(offs[-1])

    def make(shape, sigma=1.0):
        x = (sigma * rng.standard_normal(shape)).astype(np.float32)
        return kvsynth.f32_to_bf16_bits(x) if dtype == "bf16" else x
    K, V, Q = make((1, rows, d)), make((1, rows, d), 2.0), make((1, L, H * group, d))
    record = group * (d + 2)
    workspace = torch.full((L * H * 64 * record,), float("nan"), device="cuda")
    scale = float(1.0 / np.sqrt(d))
    out = fc.decode_attention(pu.to_torch(Q, dtype), pu.to_torch(K, dtype), pu.to_torch(V, dtype), H,
                              torch.from_numpy(budgets.astype(np.int32)[None]).cuda(),
                              torch.from_numpy(offs[None]).cuda(), rows, scale, workspace=workspace.view(torch.uint8))
    splits = 1024 // (L * H)
    written = ~torch.isnan(workspace.view(-1, record)[:, 0]).cpu().numpy()
    for u in range(L * H):
        pieces = min(splits, max(1, -(-int(budgets[u // H]) // 128)))
        assert np.array_equal(written[u * splits:(u + 1) * splits], np.arange(splits) < pieces), u
    assert not written[L * H * splits:].any()
    want = ref.decode_attention(Q[0], K[0], V[0], dtype, budgets, H, scale)
    err = np.abs(out.cpu().numpy()[0] - want).max()
    assert err <= 5e-5 * float(np.abs(ref.widen(V, dtype)).max())


# A launch of up to 512 column pairs spreads each grid transform over more threads (lengths 96 to 1536 with a factor of 3,
# 3072 and 4096); the layers' units together make more than that
@pytest.mark.parametrize("n,r,dtype", [(512, 52, "f32"), (1023, 109, "bf16"), (2048, 210, "bf16"), (4099, 410, "bf16"), (8191, 820, "bf16"),
                                       (16384, 1639, "bf16"), (20001, 2300, "bf16")])
def test_scores_of_small_launches_are_the_same_bits(n, r, dtype):
    import paper_2511_16786_amd as fc
    gen = torch.Generator(device="cuda").manual_seed(n)
    L, H, d = 5, 1, 128
    K, V = (torch.randn((1, L, H, n, d), generator=gen, device="cuda").to(torch.float32 if dtype == "f32" else torch.bfloat16)
            for _ in range(2))
    all_at_once = fc.Compressor(K, r, fc.total_budget(L, n, 0.2))
    all_at_once.run_score(K, V)
    one = fc.Compressor(K[:, :1], r, fc.total_budget(1, n, 0.2))
    for _ in range(2):                                           # (nothing is left behind for the next call)
        for l in range(L):
            one.run_score(K[:, l:l + 1], V[:, l:l + 1])
            assert torch.equal(one.scores[:, 0], all_at_once.scores[:, l])
            assert torch.equal(one.energy[:, 0], all_at_once.energy[:, l])
    assert fc.workspace_error(one.workspace) == 0


# One, two or four tiles of the grid to a wave by the launch's size: a tile takes its steps in an order of its own, that of its
# group of four, with fewer and with more than two tokens for each grid point and a last group that is not full
@pytest.mark.parametrize("n,r,heads", [(4099, 410, 24), (4099, 410, 90), (3001, 700, 90), (1000, 54, 300), (20001, 1000, 60)])
@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_scores_by_the_tiles_of_a_wave_are_the_same_bits(n, r, heads, dtype):
    import paper_2511_16786_amd as fc
    gen = torch.Generator(device="cuda").manual_seed(n + heads)
    K, V = (torch.randn((1, 1, heads, n, 128), generator=gen, device="cuda").to(torch.float32 if dtype == "f32" else torch.bfloat16)
            for _ in range(2))
    comp = fc.Compressor(K, r, fc.total_budget(1, n, 0.2))
    comp.run_score(K, V)
    one = fc.Compressor(K[:, :, :1], r, fc.total_budget(1, n, 0.2))
    for h in (0, heads // 2, heads - 1):
        one.run_score(K[:, :, h:h + 1], V[:, :, h:h + 1])
        assert torch.equal(one.scores[:, :, 0], comp.scores[:, :, h])
        assert torch.equal(one.energy[:, :, 0], comp.energy[:, :, h])


# Blocks of a window's tiles with a wave each (16, 13, 9, 6, 3 and 1 tiles to a window, last windows of every length) for 1, 2 and 4
# waves a unit, one unit, a few and more than fit; together the units make launches of whole windows
@pytest.mark.parametrize("n,r", [(1600, 40), (1381, 65), (1000, 85), (700, 66), (690, 130), (2310, 140), (600, 260)])
@pytest.mark.parametrize("d,dtype", [(64, "bf16"), (128, "bf16"), (256, "bf16"), (72, "f32"), (32, "f32")])
def test_blocks_of_a_windows_tiles_are_the_same_bits(n, r, d, dtype):
    import paper_2511_16786_amd as fc
    _scores_and_energies_follow_the_oracle(n, r, d, dtype, 3)
    gen = torch.Generator(device="cuda").manual_seed(n + d)
    heads = 170
    K, V = (torch.randn((1, 1, heads, n, d), generator=gen, device="cuda").to(torch.float32 if dtype == "f32" else torch.bfloat16)
            for _ in range(2))
    scale = 2.0 ** torch.randint(-12, 12, (n, 1), generator=gen, device="cuda")   # (sums that no order leaves exact)
    K, V = K * scale.to(K.dtype), V * scale.flip(0).to(V.dtype)
    comp = fc.Compressor(K, r, fc.total_budget(1, n, 0.2))
    comp.run_score(K, V)
    for first, count in ((0, 1), (5, 7), (33, 40)):
        part = fc.Compressor(K[:, :, :count], r, fc.total_budget(1, n, 0.2))
        part.run_score(K[:, :, first:first + count], V[:, :, first:first + count])
        assert torch.equal(part.scores, comp.scores[:, :, first:first + count])
        assert torch.equal(part.energy, comp.energy[:, :, first:first + count])


# The kept energy is added up per thread of the transform in 32 bits, of at most 48 points with two products each, and differently by
# the launch that spreads a transform over more threads; then in 64 bits.  The points are the same bits.
@pytest.mark.parametrize("n,r,dtype", [(512, 52, "f32"), (1023, 109, "bf16"), (2048, 210, "bf16"), (4099, 410, "bf16"), (8191, 820, "bf16"),
                                       (16384, 1639, "bf16"), (20001, 2300, "bf16")])
def test_kept_energies_of_small_launches(n, r, dtype):
    import paper_2511_16786_amd as fc
    gen = torch.Generator(device="cuda").manual_seed(n)
    L, H, d = 5, 1, 128
    K, V = (torch.randn((1, L, H, n, d), generator=gen, device="cuda").to(torch.float32 if dtype == "f32" else torch.bfloat16)
            for _ in range(2))
    kept = []
    for part in (L, 1):
        comp = fc.Compressor(K[:, :part], r, fc.total_budget(part, n, 0.2))
        for l in range(0, L, part):
            comp.run_score(K[:, l:l + part], V[:, l:l + part])
            low = torch.empty((1, part, H, 2), dtype=torch.float64, device="cuda")
            fc.lowpass_energy(comp.desc, r, comp.path, comp.workspace, low)
            kept.append(low)
            # total less kept is what was removed (Parseval)
            total, removed = comp.energy[..., 2:], comp.energy[..., :2]
            assert bool(((total - low - removed).abs() <= 2e-5 * total).all())
    assert float(((torch.cat(kept[1:], 1) - kept[0]).abs() / kept[0]).max()) <= 2 * 96 * 2.0 ** -24


@pytest.mark.parametrize("n,r,d", [(300, 33, 64), (4096, 1639, 128)])
def test_workspaces_at_any_multiple_of_256(n, r, d):
    import paper_2511_16786_amd as fc
    gen = torch.Generator(device="cuda").manual_seed(n)
    K, V = (torch.randn((1, 3, 2, n, d), generator=gen, device="cuda").to(torch.bfloat16) for _ in range(2))
    desc = fc.describe(K)
    path = fc.resolve_path(desc, r)
    size = fc.workspace_bytes(desc, r, fc.realisation(desc, r, path))
    out = []
    for at in (0, 256, 512, 768):
        held = torch.full((size + 1024 + 4096,), 0x5A, dtype=torch.uint8, device="cuda")
        at += -held.data_ptr() % 512
        workspace = held[at:at + size]
        fc.prepare(desc, r, path, workspace)
        scores = torch.empty((1, 3, 2, n), device="cuda")
        energy = torch.empty((1, 3, 2, 4), dtype=torch.float64, device="cuda")
        fc.score(K, V, desc, r, path, scores, energy, workspace)
        assert fc.workspace_error(workspace) == 0
        assert bool((held[:at] == 0x5A).all()) and bool((held[at + size:] == 0x5A).all())     # (nothing beyond its size)
        out.append((scores, energy))
    for scores, energy in out[1:]:
        assert torch.equal(scores, out[0][0]) and torch.equal(energy, out[0][1])


def test_calls_go_to_the_current_stream():
    from paper_2511_16786_amd import binding
    side = torch.cuda.Stream()
    for stream in (torch.cuda.default_stream(), side, torch.cuda.default_stream()):
        with torch.cuda.stream(stream):
            assert binding._stream() == torch.cuda.current_stream().cuda_stream == stream.cuda_stream


def _scores_and_energies_follow_the_oracle(n, r, d, dtype, heads):
    import paper_2511_16786_amd as fc
    rng = np.random.default_rng(n + r + d)
    K, V = (_smooth_plus_noise(rng, (1, 1, heads, n, d), dtype) for _ in range(2))
    want = ref.score(K, V, dtype, r, route="fast")
    comp = fc.Compressor(pu.to_torch(K, dtype), r, ref.total_budget(1, n, 0.2))
    comp.run_score(pu.to_torch(K, dtype), pu.to_torch(V, dtype))
    torch.cuda.synchronize()
    assert fc.workspace_error(comp.workspace) == 0
    pu.check_scores(comp.scores.cpu().numpy(), want["score"], pu.unit_power(ref.widen(K, dtype), ref.widen(V, dtype)))
    e = comp.energy.cpu().numpy()
    assert np.allclose(e[..., 2:], want["energy"][..., 2:], rtol=1e-5)
    assert np.all(np.abs(e[..., :2] - want["energy"][..., :2]) <= 1e-4 * want["energy"][..., :2] + 1e-7 * want["energy"][..., 2:])


# Windows of the residual kernel that hold a single tile (fewer than 1.7 tokens for each grid point), with more of them than
# workgroups, the last unit's set not full and the last tile not whole
@pytest.mark.parametrize("n,r,d,heads", [(4000, 1400, 64, 14), (2047, 1000, 128, 21), (2050, 880, 256, 18)])
@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_windows_of_a_single_tile(n, r, d, heads, dtype):
    _scores_and_energies_follow_the_oracle(n, r, d, dtype, heads)


# fp32 rows come in pieces of four columns: 1, 2, 4 and 8 waves per unit, whole and partly filled, tensors that meet inside a
# wave and between two; few units (a workgroup's waves take a unit's parts side by side) and more
@pytest.mark.parametrize("d", [8, 32, 40, 64, 104, 128, 136, 248, 256])
@pytest.mark.parametrize("n,r,heads", [(1500, 150, 3), (3100, 150, 37)])
def test_fp32_rows_of_every_width(d, n, r, heads):
    _scores_and_energies_follow_the_oracle(n, r, d, "f32", heads)


# The residual kernel's sums over a wave that holds K alone, V alone, both or some of either, and its next segments: an XCD's
# rectangle narrower and wider than its workgroups are many
@pytest.mark.parametrize("d", [16, 72, 96, 128, 200])
@pytest.mark.parametrize("n,r,heads", [(3100, 150, 70), (16000, 3000, 11)])
def test_bf16_segments_of_every_width(d, n, r, heads):
    _scores_and_energies_follow_the_oracle(n, r, d, "bf16", heads)


# The grids of 24576, 32768 and 36864 points at the fewest and most modes and tokens they take, and just beyond
@pytest.mark.parametrize("n,r,d,heads", [(20480, 10240, 16, 2), (20483, 10241, 64, 1), (47568, 10894, 8, 3), (28087, 14043, 24, 1),
                                         (28088, 14044, 16, 2), (66001, 14100, 64, 1), (37449, 18724, 8, 3), (65536, 18725, 16, 1),
                                         (42130, 21065, 8, 3), (66001, 21065, 8, 1), (65536, 21066, 16, 1), (24576, 9453, 16, 2),
                                         (24575, 9453, 8, 1), (30000, 9452, 8, 1)])
@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_scores_at_the_longest_grids(n, r, d, heads, dtype):
    import paper_2511_16786_amd as fc
    desc = fc.describe(torch.empty((1, 1, heads, n, d), dtype=torch.bfloat16 if dtype == "bf16" else torch.float32))
    assert (fc.realisation(desc, r) == fc.binding.PATHS["resample"]) == ((r, n) not in ((21066, 65536), (9453, 24575), (9452, 30000)))
    _scores_and_energies_follow_the_oracle(n, r, d, dtype, heads)


# What they replace is 2.3e-7 to 4.3e-7 (the basis) and 6.2e-8 to 6.5e-8 (the streaming transform) from 64 bits
@pytest.mark.parametrize("n,r", [(20490, 10240), (29435, 10759), (30720, 14300), (37449, 18724), (60000, 14044), (42131, 21065)])
@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_scores_at_the_longest_grids_are_as_good_as_64_bits(n, r, dtype):
    """White columns: a transform's sqrt(2 log2 M) roundings of 2.5e-8 count by what the removed modes keep of them, at most
    half here; with the scores' own rounding and the sums' 7.8e-8 at the highest cut-off, for which a quarter more is left."""
    import paper_2511_16786_amd as fc
    gen = torch.Generator(device="cuda").manual_seed(n)
    K, V = (torch.randn((1, 1, 1, n, 64), generator=gen, device="cuda").to(
        torch.bfloat16 if dtype == "bf16" else torch.float32) for _ in range(2))
    comp = fc.Compressor(K, r, ref.total_budget(1, n, 0.2))
    comp.run_score(K, V)
    s = sum(_residual64(X, r).pow(2).sum(-1) for X in (K, V)) / 64
    assert float((comp.scores.double() - s).norm() / s.norm()) <= 1e-7


# Short sequences, whose tiles and windows are fewer than XCDs or a few more, of few units and of many
@pytest.mark.parametrize("n,r,d,heads", [(300, 20, 64, 3), (512, 50, 128, 33), (700, 70, 64, 90), (1024, 91, 64, 140), (1938, 220, 128, 31),
                                         (4096, 410, 32, 60)])
@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_short_sequences(n, r, d, heads, dtype):
    _scores_and_energies_follow_the_oracle(n, r, d, dtype, heads)


# Small launches copy the rows in the selection's workgroups: as many for an index set as its budget takes of them, at the sizes of
# every such kernel, for 1 to 64 sets, budgets of one row beside whole layers, and one set more than that
@pytest.mark.parametrize("n,B,L,H", [(1024, 1, 1, 1), (513, 3, 1, 5), (1025, 2, 4, 8), (4096, 2, 7, 2), (2047, 1, 64, 1), (2050, 1, 13, 5),
                                     (5000, 1, 3, 2), (16384, 2, 2, 3)])
@pytest.mark.parametrize("shared", [False, True])
def test_rows_copied_by_the_selection(n, B, L, H, shared):
    import paper_2511_16786_amd as fc
    d, page = 24, 64
    rng = np.random.default_rng(n + L)
    K, V = (rng.integers(0, 0x7F80, (B, L, H, n, d)).astype(np.uint16) for _ in range(2))
    scores = rng.integers(0, 3 + n // 4, (B, L, H, n)).astype(np.float32)
    budgets = rng.integers(1, max(2, n // 16), (B, L))
    if L > 1:
        budgets[:, 0], budgets[:, -1] = n // 2, 1
    budgets[1:, 0] += budgets[0].sum() - budgets[1:].sum(1)               # (sequences keep as many rows)
    assert budgets.min() >= 1 and budgets.max() <= n
    offs = np.stack([ref.layer_offsets(x, H) for x in budgets])
    rows = int(offs[0, -1])
    Kt, Vt = pu.to_torch(K, "bf16"), pu.to_torch(V, "bf16")
    s_t, b_t, o_t = (torch.from_numpy(x).cuda() for x in (scores, budgets.astype(np.int32), offs))
    idx = torch.full((B, rows), -1, dtype=torch.int32, device="cuda")
    Ko, Vo = (torch.zeros((B, rows, d), dtype=Kt.dtype, device="cuda") for _ in range(2))
    desc = fc.describe(Kt)
    fc.select_gather(Kt, Vt, desc, s_t, b_t, o_t, rows, idx, Ko, Vo, shared=shared)
    reach = -(-n // page) - 1                                             # (rows of a last page that is not there are left out)
    table = rng.permutation(B * L * H * reach).astype(np.int32).reshape(B, L, H, reach)
    Kc, Vc = (torch.zeros((B * L * H * reach, page, d), dtype=Kt.dtype, device="cuda") for _ in range(2))
    fc.select_gather_paged(Kt, Vt, desc, s_t, b_t, o_t, rows, torch.empty_like(idx), torch.from_numpy(table).cuda(), page, Kc, Vc,
                           shared=shared)
    paged = [np.zeros(Kc.shape, dtype=K.dtype) for _ in range(2)]
    for b in range(B):
        want = ref.select_gather(K[b], V[b], scores[b], budgets[b], shared=shared)
        assert np.array_equal(idx[b].cpu().numpy(), want["idx"])
        for got, name, out in ((Ko, "K_out", paged[0]), (Vo, "V_out", paged[1])):
            assert np.array_equal(pu.rows_to_numpy(got, "bf16")[b], want[name])
            for l in range(L):
                for h in range(H):
                    at = offs[b, l] + h * budgets[b, l]
                    for j in range(min(int(budgets[b, l]), reach * page)):
                        out[table[b, l, h, j // page], j % page] = want[name][at + j]
    assert np.array_equal(pu.rows_to_numpy(Kc, "bf16"), paged[0]) and np.array_equal(pu.rows_to_numpy(Vc, "bf16"), paged[1])


# ... and of launches on both sides of the most column pairs that are spread: 512, 1024 (768 and 3072 points) and 2048 (384), by
# units of 32 pairs
@pytest.mark.parametrize("n,r,most", [(8191, 820, 512), (4099, 410, 1024), (16384, 1639, 1024), (2048, 210, 2048)])
def test_scores_on_both_sides_of_the_spread_launches(n, r, most):
    import paper_2511_16786_amd as fc
    gen = torch.Generator(device="cuda").manual_seed(n)
    units, d = most // 32 + 1, 32
    K, V = (torch.randn((1, units, 1, n, d), generator=gen, device="cuda").to(torch.bfloat16) for _ in range(2))
    every = fc.Compressor(K, r, fc.total_budget(units, n, 0.2))
    every.run_score(K, V)
    fewer = fc.Compressor(K[:, :-1], r, fc.total_budget(units - 1, n, 0.2))
    fewer.run_score(K[:, :-1], V[:, :-1])
    assert torch.equal(fewer.scores, every.scores[:, :-1]) and torch.equal(fewer.energy, every.energy[:, :-1])
    assert fc.workspace_error(every.workspace) == 0 and fc.workspace_error(fewer.workspace) == 0


# Tables that reach 128 rows make one piece of every unit, which needs no merge; tables that reach further make the same pieces of the
# same budgets, and merge them
@pytest.mark.parametrize("d,group", [(64, 4), (128, 7)])
@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_decode_of_single_pieces_is_the_merged_one(dtype, d, group):
    import paper_2511_16786_amd as fc
    B, L, H, page = 2, 3, 2, 64
    gen = torch.Generator(device="cuda").manual_seed(d)
    dt = torch.float32 if dtype == "f32" else torch.bfloat16
    Q = torch.randn((B, L, H * group, d), generator=gen, device="cuda").to(dt)
    units = B * L * H
    K, V = (torch.randn((units * 2, page, d), generator=gen, device="cuda").to(dt) for _ in range(2))
    budgets = torch.tensor([[128, 1, 77], [64, 0, 33]], dtype=torch.int32, device="cuda")
    short = torch.randperm(units * 2, generator=gen, device="cuda").to(torch.int32).view(B, L, H, 2)
    long = torch.cat((short, torch.full((B, L, H, 3), -1, dtype=torch.int32, device="cuda")), 3).contiguous()
    out = [fc.decode_attention_paged(Q, K, V, H, budgets, t, d ** -0.5) for t in (short, long)]
    assert torch.equal(out[0], out[1]) and bool((out[0][1, 1] == 0).all()) and bool(torch.isfinite(out[0]).all())
    for b in range(B):
        for l in range(L):
            k = int(budgets[b, l])
            for h in range(H if k else 0):
                rows = [x[short[b, l, h].long()].reshape(-1, d)[:k].double() for x in (K, V)]
                p = torch.softmax(Q[b, l, h * group:(h + 1) * group].double() @ rows[0].T * d ** -0.5, -1)
                want = p @ rows[1]
                assert float((out[0][b, l, h * group:(h + 1) * group] - want).abs().max()) <= 5e-5 * float(rows[1].abs().max())


def _softmax64(Q, rows_k, rows_v, scale):
    return torch.softmax(Q.double() @ rows_k.double().T.contiguous() * scale, -1) @ rows_v.double()


# Single pieces of caches larger than the last-level cache: more than 1024 units, layers that keep nothing, little and much, packed and
# through tables whose pool is as large
@pytest.mark.parametrize("dtype,d,group", [("bf16", 128, 7), ("f32", 64, 4)])
def test_decode_of_single_pieces_of_large_caches(dtype, d, group):
    import paper_2511_16786_amd as fc
    B, L, H, page = 8, 36, 4, 64
    gen = torch.Generator(device="cuda").manual_seed(d)
    rng = np.random.default_rng(d)
    dt = torch.float32 if dtype == "f32" else torch.bfloat16
    of_layers = np.concatenate(([0, 1, 63, 64, 2500], rng.integers(300, 620, L - 5)))
    budgets = np.stack([rng.permutation(of_layers) for _ in range(B)])
    offs = np.stack([ref.layer_offsets(x, H) for x in budgets])
    rows = int(offs[0, -1])
    assert 2 * B * rows * d * (4 if dtype == "f32" else 2) > 256e6 and B * L * H > 1024
    Q = torch.randn((B, L, H * group, d), generator=gen, device="cuda").to(dt)
    K, V = (torch.randn((B, rows, d), generator=gen, device="cuda").to(dt) for _ in range(2))
    b_t, o_t = torch.from_numpy(budgets.astype(np.int32)).cuda(), torch.from_numpy(offs).cuda()
    packed = fc.decode_attention(Q, K, V, H, b_t, o_t, rows, d ** -0.5)
    # the same rows in pages of a shuffled pool, which holds what the budgets take
    pages = -(-budgets // page)
    table = np.full((B, L, H, int(pages.max())), -1, dtype=np.int32)
    order, at = rng.permutation(int(pages.sum()) * H).astype(np.int32), 0
    Kp, Vp = (torch.zeros((len(order), page, d), dtype=dt, device="cuda") for _ in range(2))
    for b in range(B):
        for l in range(L):
            for h in range(H):
                k, n = int(budgets[b, l]), int(pages[b, l])
                table[b, l, h, :n] = order[at:at + n]
                at += n
                where = torch.from_numpy(table[b, l, h, :n].astype(np.int64)).cuda()
                first = int(offs[b, l]) + h * k
                for src, dst in ((K, Kp), (V, Vp)):
                    x = torch.zeros((n * page, d), dtype=dt, device="cuda")
                    x[:k] = src[b, first:first + k]
                    dst[where] = x.view(n, page, d)
    paged = fc.decode_attention_paged(Q, Kp, Vp, H, b_t, torch.from_numpy(table).cuda(), d ** -0.5)
    assert bool(torch.isfinite(packed).all()) and bool(torch.isfinite(paged).all())
    for b in (0, 3, B - 1):
        for l in range(L):
            k = int(budgets[b, l])
            for h in range(H):
                q = Q[b, l, h * group:(h + 1) * group]
                got = [x[b, l, h * group:(h + 1) * group] for x in (packed, paged)]
                if k == 0:
                    assert all(bool((x == 0).all()) for x in got)
                    continue
                first = int(offs[b, l]) + h * k
                want = _softmax64(q, K[b, first:first + k], V[b, first:first + k], d ** -0.5)
                for x in got:
                    assert float((x - want).abs().max()) <= 5e-5 * float(V[b, first:first + k].abs().max())


# Packed sequences of no more than 128 rows a head make one piece of every unit as well
@pytest.mark.parametrize("budgets", [[128], [1, 0, 127], [40, 41, 47]])
@pytest.mark.parametrize("dtype,d,group", [("bf16", 128, 7), ("bf16", 64, 1), ("f32", 128, 8)])
def test_decode_of_packed_single_pieces(budgets, dtype, d, group):
    import paper_2511_16786_amd as fc
    B, L, H = 3, len(budgets), 2
    gen = torch.Generator(device="cuda").manual_seed(d + L)
    dt = torch.float32 if dtype == "f32" else torch.bfloat16
    offs = ref.layer_offsets(np.array(budgets), H)
    rows = int(offs[-1])
    Q = torch.randn((B, L, H * group, d), generator=gen, device="cuda").to(dt)
    K, V = (torch.randn((B, rows, d), generator=gen, device="cuda").to(dt) for _ in range(2))
    b_t = torch.tensor([budgets] * B, dtype=torch.int32, device="cuda")
    got = fc.decode_attention(Q, K, V, H, b_t, torch.from_numpy(np.stack([offs] * B)).cuda(), rows, d ** -0.5)
    for b in range(B):
        for l, k in enumerate(budgets):
            for h in range(H):
                x = got[b, l, h * group:(h + 1) * group]
                if k == 0:
                    assert bool((x == 0).all())
                    continue
                first = int(offs[l]) + h * k
                want = _softmax64(Q[b, l, h * group:(h + 1) * group], K[b, first:first + k], V[b, first:first + k], d ** -0.5)
                assert float((x - want).abs().max()) <= 5e-5 * float(V[b, first:first + k].abs().max())


# Units of three and of five to eight parts, two with empty lanes: parts side by side in workgroups of three to eight waves, one segment for
# each wave and more, and in turn, of windows of a single tile, of a few and of blocks
@pytest.mark.parametrize("n,r", [(1500, 150), (690, 60), (2050, 900), (8200, 3500)])
@pytest.mark.parametrize("d,dtype", [(40, "f32"), (72, "f32"), (136, "f32"), (192, "f32"), (224, "f32"), (256, "f32"), (136, "bf16"), (192, "bf16")])
def test_parts_side_by_side_and_in_turn_are_the_same_bits(n, r, d, dtype):
    import paper_2511_16786_amd as fc
    if n < 8000:
        _scores_and_energies_follow_the_oracle(n, r, d, dtype, 3)
    gen = torch.Generator(device="cuda").manual_seed(n + d)
    heads = 130 if n < 8000 else 30
    K, V = (torch.randn((1, 1, heads, n, d), generator=gen, device="cuda").to(torch.float32 if dtype == "f32" else torch.bfloat16)
            for _ in range(2))
    every = fc.Compressor(K, r, fc.total_budget(1, n, 0.2))
    every.run_score(K, V)
    for first, count in ((0, 1), (3, 3), (7, 20)):
        part = fc.Compressor(K[:, :, :count], r, fc.total_budget(1, n, 0.2))
        part.run_score(K[:, :, first:first + count], V[:, :, first:first + count])
        assert torch.equal(part.scores, every.scores[:, :, first:first + count])
        assert torch.equal(part.energy, every.energy[:, :, first:first + count])
    assert fc.workspace_error(every.workspace) == 0
