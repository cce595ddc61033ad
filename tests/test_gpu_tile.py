"""The two-dimensional-tile kernel (CNN_K_IGEMM, variants from 3000 on): every
form of its staging, at the edges of its tiles, against the fp64 oracle."""
import numpy as np
import pytest

import oracle
from paper_2105_13480_amd import cnn, inputs

from gpu_helpers import TOL, errors, run, say, variant_plan

pytestmark = pytest.mark.gpu

MODES = {"f32": cnn.CNN_F32, "bf16": cnn.CNN_BF16, "bf16_obf16": cnn.CNN_BF16_OBF16}

# (Nb, Nc, Nk, Nw, Nh, Nr, Ns, sw, sh)
SHAPES = [
    (2, 17, 33, 20, 75, 3, 3, 1, 1),    # column bands, one channel in the last stage
    (3, 16, 64, 7, 7, 3, 3, 1, 1),      # tiles across images, whole channels
    (1, 5, 3, 6, 300, 3, 3, 1, 1),      # rows wider than a tile, fewer channels than a stage
    (2, 33, 70, 9, 14, 3, 3, 2, 2),     # columns by parity
    (2, 24, 40, 5, 9, 3, 3, 3, 3),      # stride 3: position pairs
    (1, 31, 45, 4, 2, 3, 3, 1, 1),      # four columns: pairs
    (2, 65, 66, 11, 13, 1, 1, 1, 1),    # 1x1, odd rows, odd Ker elements
    (3, 79, 131, 9, 17, 1, 1, 2, 2),    # 1x1 gathered at stride 2
    (2, 72, 40, 6, 10, 1, 1, 2, 3),     # 1x1 gathered at stride 3, rows squeezed
    (2, 19, 21, 9, 11, 1, 7, 1, 1),     # runtime stencils: 7 taps, odd
    (2, 21, 37, 9, 11, 7, 1, 2, 2),     # 1 wide, gathered, 7 rows
    (2, 18, 35, 10, 12, 3, 2, 2, 1),    # 6 taps
    (1, 23, 50, 12, 21, 5, 5, 1, 1),    # 25 taps
    (2, 16, 20, 8, 9, 4, 4, 2, 2),      # 16 taps, even stencil at stride 2
    (1, 9, 34, 8, 10, 7, 7, 2, 2),      # 49 taps
    (2, 20, 24, 6, 15, 2, 3, 3, 1),     # rows between reads not staged
    (1, 1, 1, 1, 2, 1, 1, 1, 1),        # the smallest
    (1, 3, 1, 1, 8, 1, 1, 1, 1),        # one row of one vector, three Ker elements
]


# No instantiation fits: the Ker items of 49 fp32 taps a stage.
NO_TILE = {("f32", (1, 9, 34, 8, 10, 7, 7, 2, 2))}


def _ints(dims, mode, seed):
    return inputs.make_arrays(*dims, "f32" if mode == "f32" else "bf16", seed_in=seed,
                              seed_ker=seed + 1, in_dist=("int", -2, 2), ker_dist=("int", -2, 2))


def _tile_plans(dims, mode):
    """The tile plans of a problem for a full and for a small GPU budget (few
    CUs: the largest tiles)."""
    seen, out = set(), []
    for cus in (256, 2):
        for c in cnn.plan_candidates(cnn.problem(*dims), MODES[mode], cnn.budget(cus=cus)):
            if c.kernel == cnn.K_IGEMM and 3000 <= c.variant < 3300 and (c.variant, c.kc) not in seen:
                seen.add((c.variant, c.kc))
                out.append(c)
    return out


def _tiling(dims, mode, tk, tp, tc):
    """The plan of a tiling the caller names, None if there is none."""
    try:
        return cnn.plan_tiles(cnn.problem(*dims), MODES[mode], cnn.K_IGEMM, tk, tp, tc)
    except cnn.CnnError:
        return None


def _all_tile_plans(dims, mode):
    """The tile plans of a problem, also by tilings that the selector leaves out."""
    plans = {}
    for v in cnn.variants():
        if v.kernel == cnn.K_IGEMM and 3000 <= v.variant < 3300 and v.dtype == MODES[mode]:
            pl = variant_plan(dims, v.dtype, v.kernel, v.tk, v.tp, v.tc, v.variant) or \
                _tiling(dims, mode, v.tk, v.tp, v.tc)
            if pl is not None and 3000 <= pl.variant < 3300:
                plans[pl.variant] = pl
    return list(plans.values())


@pytest.mark.parametrize("mode", list(MODES))
@pytest.mark.parametrize("dims", SHAPES, ids=str)
def test_tile_exact_integers(dims, mode):
    """Integer inputs: every sum exact in fp32, so bit-exact in fp32 Out and
    its rounding in bf16 Out."""
    In, Ker = _ints(dims, mode, seed=sum(dims))
    want = oracle.conv(In, Ker, dims[7], dims[8])
    if mode == "bf16_obf16":
        want = oracle.widen(inputs.f32_to_bf16_bits(want.astype(np.float32)))
    plans = _tile_plans(dims, mode)
    if not plans:  # sums the selector leaves to the fp32 units: by their tilings
        plans = _all_tile_plans(dims, mode)
    assert plans or (mode, dims) in NO_TILE
    for pl in plans:
        say(f"[tile] dims={dims} mode={mode} v{pl.variant} rows={pl.kc} tp={pl.tp} grid={pl.grid}")
        got = run(In, Ker, dims[7], dims[8], mode, plan=pl)
        assert np.array_equal(got, want), (pl.variant, pl.kc)


@pytest.mark.parametrize("dims", [(2, 70, 70, 13, 21, 3, 3, 1, 1), (2, 130, 40, 9, 11, 1, 1, 2, 2),
                                  (1, 40, 33, 12, 12, 5, 5, 1, 1)] +
                         [(2, nc, 64, 40, 40, r, r, 1, 1) for r in (1, 3) for nc in (1, 2, 4, 5, 9, 10, 17, 18)],
                         ids=str)
def test_tile_f32_split_error(dims):
    """fp32 as three bf16 parts, against 64 bits.  Per product the parts that
    are dropped come to at most 2^-7 2^-16 twice, less than 4 units of 2^-24;
    the leading sum rounds once per tap and 8 channels (K / 8 of them, K padded
    to whole stages of 32 channels), the small ones five times that 2^-7 smaller,
    and their sum once more.  And no more than the fp32 units' own error, also
    for short sums and few channels in the last eight (tenth: the spread of the
    2-norm over these many outputs)."""
    Nc, RS = dims[1], dims[5] * dims[6]
    bound = (-(-Nc // 32) * 4 * RS * (1 + 5 / 128) + 5) * 2.0 ** -24
    In, Ker = inputs.make_arrays(*dims, "f32", seed_in=5, seed_ker=6,
                                 in_dist=("uniform", 0.0, 1.0), ker_dist=("he",))
    want, absv = oracle.conv(In, Ker, dims[7], dims[8], with_abs=True)

    def rms(got):
        return np.linalg.norm((got - want).ravel()) / np.linalg.norm(want.ravel())

    units = run(In, Ker, dims[7], dims[8], "f32", plan=_tiling(dims, "f32", 64, 64, 8))
    plans = _all_tile_plans(dims, "f32")
    assert plans
    for pl in plans:
        say(f"[tile] f32 error dims={dims} v{pl.variant} rows={pl.kc}")
        got = run(In, Ker, dims[7], dims[8], "f32", plan=pl)
        nw, cond, _ = errors(got, want, absv)
        assert cond <= min(bound, TOL["f32"]) and nw <= TOL["f32"], (pl.variant, nw, cond)
        assert rms(got) <= 1.1 * rms(units), (pl.variant, rms(got), rms(units))


@pytest.mark.parametrize("dims", [(2, 20, 40, 9, 13, 3, 3, 1, 1), (1, 33, 34, 6, 9, 1, 1, 2, 2),
                                  (1, 18, 20, 8, 9, 4, 2, 1, 2)], ids=str)
@pytest.mark.parametrize("case", ["inf", "nan", "lowest", "overflow", "tiny", "subnormal"])
def test_tile_f32_outside_the_split(dims, case):
    """Values that three bf16 parts do not hold: infinities and NaN reach
    exactly the outputs that the direct fp32 kernel's reach, the type's lowest
    value stays finite, products that overflow are infinite and not NaN, and inputs near the bottom of the range keep fp32's
    relative accuracy."""
    In, Ker = inputs.make_arrays(*dims, "f32", seed_in=8, seed_ker=9,
                                 in_dist=("uniform", 0.25, 1.0), ker_dist=("he",))
    In = In.copy()
    if case == "inf":
        In[0, 3, 2, 4], In[-1, 5, 1, 1] = np.inf, -np.inf
    elif case == "nan":
        In[0, 3, 2, 4] = np.nan
    elif case == "lowest":
        In[0, 3, 2, 4] = np.finfo(np.float32).min
    elif case == "overflow":  # (1e25 1e25 > 2^144: the lowest parts' products too)
        In *= np.float32(1e25)
        Ker = np.abs(Ker) * np.float32(1e25)
    elif case == "tiny":
        In *= np.float32(1e-34)
    else:  # the first image's outputs are a subnormal channel's alone
        In[0, :3], In[0, 4:] = 0, 0
        In[0, 3] *= np.float32(1e-40)
    prob = cnn.problem(*dims)
    say(f"[tile] f32 {case} dims={dims}: direct kernel")
    ref = run(In, Ker, dims[7], dims[8], "f32", plan=cnn.plan_tiles(prob, cnn.CNN_F32, cnn.K_DIRECT))
    assert case != "overflow" or np.isposinf(ref).all()
    # each output against its own sum of |In Ker|, and the least number a product
    scale = 1e-5 * oracle.conv(np.where(np.isfinite(In), np.abs(In), 0), np.abs(Ker), dims[7], dims[8])
    scale += dims[1] * dims[5] * dims[6] * 2.0 ** -149
    plans = _tile_plans(dims, "f32")
    assert plans
    for pl in plans:
        say(f"[tile] f32 {case} dims={dims} v{pl.variant} rows={pl.kc}")
        got = run(In, Ker, dims[7], dims[8], "f32", plan=pl)
        assert np.array_equal(np.isnan(got), np.isnan(ref)), pl.variant
        assert np.array_equal(np.isinf(got), np.isinf(ref)), pl.variant
        fine = np.isfinite(ref)
        assert np.array_equal(got[np.isinf(ref)], ref[np.isinf(ref)])
        assert (np.abs(got[fine] - ref[fine]) <= scale[fine]).all(), pl.variant


@pytest.mark.parametrize("dims", [(2, 20, 40, 9, 13, 3, 3, 1, 1), (2, 33, 34, 6, 9, 1, 1, 2, 2),
                                  (2, 18, 20, 8, 9, 4, 2, 1, 2)], ids=str)
@pytest.mark.parametrize("case", ["weight", "channel", "alone", "subnormal alone", "edge", "parts",
                                  "products"])
def test_tile_f32_small_values(dims, case):
    """Values below 2^-102, whose parts are incomplete, and products below the
    least normal number keep fp32's accuracy in every output, also where they
    decide it: relative to its own sum of |In Ker| within the bound of the split
    (one unit of 2^-24 more for what the parts of small values may lose), plus a
    unit of the smallest number per product."""
    Nc, RS = dims[1], dims[5] * dims[6]
    In, Ker = inputs.make_arrays(*dims, "f32", seed_in=31, seed_ker=32,
                                 in_dist=("uniform", 0.25, 1.0), ker_dist=("he",))
    In, Ker = In.copy(), Ker.copy()
    if case == "weight":         # one small weight among ordinary ones
        Ker[0, 0, 0, 0] = 1e-35
    elif case == "channel":      # one channel that hardly counts
        In[:, 3] *= np.float32(1e-36)
    elif case == "alone":        # an image whose outputs are its small values' alone
        In[-1] *= np.float32(1e-36)
        In[-1, 5:] = 0
    elif case == "subnormal alone":
        In[-1] = 0
        In[-1, 3] = np.float32(3e-41)
    elif case == "edge":         # outputs on either side of where the parts are enough
        scale = np.exp2(np.linspace(-100, -70, In.shape[3])).astype(np.float32)
        In *= scale
        In[:, 2] = np.float32(1e-33)
    elif case == "parts":        # operands in range, low parts' products below 2^-126
        In *= np.float32(2.0 ** -60)
        Ker *= np.float32(2.0 ** -62)
    else:                        # the products themselves
        In *= np.float32(2.0 ** -70)
        Ker *= np.float32(2.0 ** -66)
    want, absv = oracle.conv(In, Ker, dims[7], dims[8], with_abs=True)
    units = -(-Nc // 32) * 4 * RS * (1 + 5 / 128) + 6
    plans = _all_tile_plans(dims, "f32")
    assert plans
    for pl in plans:
        say(f"[tile] f32 small values {case} dims={dims} v{pl.variant} rows={pl.kc}")
        got = run(In, Ker, dims[7], dims[8], "f32", plan=pl)
        off = np.abs(got - want) / (units * 2.0 ** -24 * absv + Nc * RS * 2.0 ** -149)
        assert off.max() <= 1, (pl.variant, off.max())


def test_tile_f32_one_small_weight_costs_nothing():
    """A weight below 2^-102 among ordinary ones does not send the layer to the
    fp32 units: 3.5 times the time when it did, 1.1 now."""
    import torch
    from gpu_helpers import out_tensor, to_gpu
    dims = (16, 64, 64, 56, 56, 3, 3, 1, 1)
    In, Ker = inputs.make_arrays(*dims, "f32", seed_in=1, seed_ker=2,
                                 in_dist=("uniform", 0.0, 1.0), ker_dist=("he",))
    pl = _tiling(dims, "f32", 64, 256, 16)
    dIn, dOut = to_gpu(In), out_tensor(*dims[:1], *dims[2:5], "f32")

    def us(k):
        best = 1e9
        for _ in range(5):
            e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            e0.record()
            for _ in range(20):
                cnn.fwd_plan(dIn, k, dOut, pl, 1, 1)
            e1.record()
            e1.synchronize()
            best = min(best, e0.elapsed_time(e1) * 50)
        return best

    small = Ker.copy()
    small[0, 0, 0, 0] = 1e-35
    say(f"[tile] f32 one small weight v{pl.variant} rows={pl.kc}")
    plain, tiny = us(to_gpu(Ker)), us(to_gpu(small))
    say(f"[tile] {plain:.1f} us, {tiny:.1f} us with one small weight")
    assert tiny <= 2 * plain, (plain, tiny)


@pytest.mark.parametrize("dims", [(1, 32, 40, 5, 300, 3, 3, 1, 1), (1, 32, 40, 3, 290, 1, 1, 1, 1)],
                         ids=str)
def test_tile_f32_bands_store_what_they_own(dims):
    """Bands of columns, the last of which overlaps its neighbour: an infinity
    in columns that only the last band reads sends that band to the fp32 units,
    and the outputs of the overlap, which the neighbour owns, keep their bits
    in every run."""
    Nh, Ns = dims[4], dims[6]
    In, Ker = inputs.make_arrays(*dims, "f32", seed_in=21, seed_ker=22,
                                 in_dist=("uniform", -1.0, 1.0), ker_dist=("he",))
    bad = In.copy()
    bad[0, 3, 1, -1] = np.inf  # read by the last output column alone
    plans = [pl for pl in _tile_plans(dims, "f32") if Nh % (pl.tp // pl.kc)]
    assert plans
    for pl in plans:
        ct = pl.tp // pl.kc
        first = Nh // ct * ct  # the last band's own columns
        assert first < Nh - Ns
        say(f"[tile] f32 bands dims={dims} v{pl.variant} rows={pl.kc} columns={ct}")
        clean = run(In, Ker, dims[7], dims[8], "f32", plan=pl)
        for _ in range(6):
            got = run(bad, Ker, dims[7], dims[8], "f32", plan=pl)
            assert np.isinf(got[..., -1]).any()
            assert np.array_equal(got[..., :first], clean[..., :first]), pl.variant


@pytest.mark.parametrize("mode", list(MODES))
@pytest.mark.parametrize("dims", [(2, 17, 33, 9, 14, 3, 3, 1, 1), (1, 33, 19, 7, 9, 1, 1, 2, 2),
                                  (1, 6, 21, 8, 11, 1, 5, 1, 1)], ids=str)
def test_tensors_at_odd_addresses(dims, mode):
    """In, Ker and Out that start one element past an aligned address, in both
    workspace-free kernels that load 16 bytes at any alignment (the tile kernel
    and the few-outputs kernel, variants 3300 on)."""
    import torch
    from gpu_helpers import out_tensor, to_gpu, to_host64
    Nb, Nc, Nk, Nw, Nh = dims[:5]
    In, Ker = _ints(dims, mode, seed=sum(dims) + 7)
    want = oracle.conv(In, Ker, dims[7], dims[8])
    if mode == "bf16_obf16":
        want = oracle.widen(inputs.f32_to_bf16_bits(want.astype(np.float32)))

    def shifted(t):
        whole = torch.zeros(t.numel() + 1, dtype=t.dtype, device="cuda")
        view = whole[1:].view(t.shape)
        view.copy_(t)
        return view

    dIn, dKer = shifted(to_gpu(In)), shifted(to_gpu(Ker))
    few = [c for c in cnn.plan_candidates(cnn.problem(*dims), MODES[mode])
           if c.kernel == cnn.K_IGEMM and 3300 <= c.variant < 3400]
    tiles = _tile_plans(dims, mode)
    assert tiles and len(few) >= 3
    for pl in tiles + few:
        dOut = shifted(out_tensor(Nb, Nk, Nw, Nh, mode))
        say(f"[tile] odd addresses dims={dims} mode={mode} v{pl.variant} rows={pl.kc}")
        cnn.fwd_plan(dIn, dKer, dOut, pl, dims[7], dims[8])
        torch.cuda.synchronize()
        assert np.array_equal(to_host64(dOut), want), pl.variant
