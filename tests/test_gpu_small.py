"""The few-outputs kernel (CNN_K_IGEMM, variants 3300 on, and the direct
channel-slice plans it runs) at the edges of its tiles, steps and chunks,
against the fp64 oracle."""
import numpy as np
import pytest

import oracle
from paper_2105_13480_amd import cnn, inputs

from gpu_helpers import run, say

pytestmark = pytest.mark.gpu

MODES = {"f32": cnn.CNN_F32, "bf16": cnn.CNN_BF16, "bf16_obf16": cnn.CNN_BF16_OBF16}

# (Nb, Nc, Nk, Nw, Nh, Nr, Ns, sw, sh)
SHAPES = [
    (1, 512, 24, 7, 7, 3, 3, 1, 1),      # 16 waves, several steps each
    (2, 33, 17, 5, 7, 3, 3, 1, 1),       # a ragged last step, one feature in the last tile
    (1, 17, 9, 4, 9, 1, 1, 2, 2),        # fewer elements than a step
    (3, 5, 7, 1, 1, 3, 3, 1, 1),         # one output an image, 45 odd Ker elements
    (1, 3, 5, 3, 40, 5, 5, 1, 2),        # rows longer than a tile
    (1, 300, 20, 20, 24, 3, 3, 1, 1),    # a chunk of the channels at a time
    (2, 2100, 18, 9, 10, 1, 1, 1, 1),    # the same, a ragged last chunk
    (1, 64, 33, 6, 6, 7, 1, 1, 3),       # tall stencil, stride 3
    (1, 1, 1, 1, 1, 1, 1, 1, 1),         # the smallest
    (1, 7, 3, 2, 3, 2, 2, 3, 3),         # stride over the stencil
]


@pytest.mark.parametrize("mode", list(MODES))
@pytest.mark.parametrize("dims", SHAPES, ids=str)
def test_small_exact_integers(dims, mode):
    """Integer inputs: every sum exact in fp32, so bit-exact in fp32 Out and
    its rounding in bf16 Out, and the last element of each tensor is used."""
    In, Ker = inputs.make_arrays(*dims, "f32" if mode == "f32" else "bf16", seed_in=sum(dims),
                                 seed_ker=sum(dims) + 1, in_dist=("int", 1, 3), ker_dist=("int", -2, 2))
    want = oracle.conv(In, Ker, dims[7], dims[8])
    if mode == "bf16_obf16":
        want = oracle.widen(inputs.f32_to_bf16_bits(want.astype(np.float32)))
    n = 0
    for v in cnn.variants():
        if v.kernel != cnn.K_IGEMM or v.variant < 3300 or v.dtype != MODES[mode]:
            continue
        try:
            pl = cnn.plan_tiles(cnn.problem(*dims), v.dtype, cnn.K_IGEMM, v.tk, v.tp, 0)
        except cnn.CnnError:
            continue  # 32 channels' rows do not fit LDS
        say(f"[small] dims={dims} mode={mode} v{pl.variant} grid={pl.grid} lds={pl.lds_bytes}")
        got = run(In, Ker, dims[7], dims[8], mode, plan=pl)
        assert np.array_equal(got, want), pl.variant
        n += 1
    assert n >= 2


@pytest.mark.parametrize("mode", ["bf16", "bf16_obf16"])
@pytest.mark.parametrize("lds", [160, 128])
def test_direct_slices(mode, lds):
    """A direct channel-slice plan names the few-outputs kernel's launch (in
    chunks of channels where the budget's LDS is smaller), and one that carries
    the 32 x 64 tile of earlier versions still runs: both equal the oracle."""
    dims = (1, 1024, 70, 7, 9, 3, 3, 1, 1)
    prob, bud = cnn.problem(*dims), cnn.budget(lds_bytes=lds * 1024)
    In, Ker = inputs.make_arrays(*dims, "bf16", seed_in=3, seed_ker=4, in_dist=("int", -2, 2),
                                 ker_dist=("int", -2, 2))
    want = oracle.conv(In, Ker, 1, 1)
    if mode == "bf16_obf16":
        want = oracle.widen(inputs.f32_to_bf16_bits(want.astype(np.float32)))
    pl = cnn.plan_tiles(prob, MODES[mode], cnn.K_SPLITC, 32, 64, 128, bud)
    assert pl.tk in (8, 16) and (pl.tc < dims[1]) == (lds < 160) and pl.lds_bytes <= lds * 1024
    # the 32 x 64 tile: slab and grid of the other channel-slice plans, 128 channels a stage
    old = cnn.Plan.from_buffer_copy(pl)
    ref = cnn.plan_tiles(prob, MODES[mode], cnn.K_SPLITC, 32, 64, 64, bud)
    old.tk, old.tp, old.tc, old.slab_rows, old.grid = 32, 64, 128, ref.slab_rows, ref.grid
    old.lds_bytes = 16 * (9 * 16 * 33 + ref.slab_rows * 11 * 17)
    for p in (pl, old):
        say(f"[small] direct slices mode={mode} v{p.variant} tk={p.tk} tc={p.tc} lds={p.lds_bytes}")
        assert np.array_equal(run(In, Ker, 1, 1, mode, plan=p), want)
