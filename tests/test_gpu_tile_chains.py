"""Whole-layer parity where every workgroup of the tiled GEMMs runs several
tiles in a row, so the copy pipeline crosses tile boundaries.  The second
product has more tiles than workgroups here (at least 17 row tiles x 16
column tiles), and its number of K steps per tile sits on either side of
the point where the next tile's first steps stop being issued together
with the current tile's last step and start being issued in stride: 5
steps (issued together) and 6 steps (in stride) with three stages, and a
four-stage kernel (MXFP8 activations, 128-element steps) with 9 steps."""
import numpy as np
import pytest

import synth
from tests.gpu_util import check_forward, require_gpu

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def dev():
    return require_gpu()


@pytest.mark.parametrize("I", [320, 384])     # bf16 second product: 5 and 6 K steps of 64
def test_bf16_chained_tiles(dev, I):
    check_forward(synth.tiny_config(3, T=600, H=4096, E=8, I=I, top_k=4))


def test_mxfp8_four_stage_chained_tiles(dev):
    # I = 1152 is a multiple of 128 but not of 256: the second product takes
    # 128-element steps on the four-stage kernel, 9 per tile
    check_forward(synth.tiny_config(9, T=600, H=4096, E=16, I=1152, top_k=4))


@pytest.mark.parametrize("n,H,I", [(3, 512, 136), (8, 512, 256), (8, 384, 128), (4, 512, 256), (4, 384, 512),
                                   (9, 512, 256), (9, 384, 128)])
def test_padded_row_blocks(dev, n, H, I):
    # bf16 (ragged K and columns too), MXFP4, fp8 and MXFP4 x MXFP8 tiles with one to four live
    # 32-row blocks, on either side of each boundary: every token picks expert
    # e with probability falling in e, so segment lengths spread over the tile;
    # the routed rows are counted to be sure
    # (fp8 at I >= 256: one intermediate code tipped to its neighbour is up to
    # 32/448 of its group's largest value, about 3.5 / 14 of the rms, which times
    # a weight of 3.5 / sqrt(I) of the output's rms is 7.7e-2 at I = 128, past
    # the format's 6e-2, and 5.5e-2 at 256)
    cfg = synth.tiny_config(n, T=700, H=H, I=I, E=16, top_k=2)
    inp = synth.make_inputs(cfg)
    lg = np.random.default_rng(3).gumbel(size=(700, 16)) + np.log(np.arange(16, 0, -1) ** 1.5)
    bias = None if inp["sel_bias"] is None else np.zeros_like(inp["sel_bias"])
    _, ref, L = check_forward(cfg, dict(inp, logits=(lg / 4).astype(np.float32), sel_bias=bias))
    assert L["block_m"] == 128
    live = {-(-int(c % 128) // 32) or 4 for c in np.bincount(ref["ids"].ravel(), minlength=16) if c}
    assert live == {1, 2, 3, 4}, live
