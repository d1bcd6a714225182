"""The reversed direction of SC layers with f = s (DC and the SC input gradient over the pair
lists) against the oracle: fields from 2^3 to 32^2, so that offsets hold from no pair to several
tiles of them and a wave's look at the offsets takes one and two steps; on extents the stride
divides and on ones that it does not but whose sites all lie in whole fields; on the dense grid and
on the table of sites.  Bounds as in the other parity tests."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

import oracle  # noqa: E402
import paper_1706_01307_amd as spc  # noqa: E402
from paper_1706_01307_amd import inputs  # noqa: E402
from tests.test_ops_gpu import _dev, _feats, _odt  # noqa: E402
from tests.test_parity_gpu import (RTOL_BF16, RTOL_F32, _say, _t, _to_np,  # noqa: E402
                                   check_features)

pytestmark = pytest.mark.gpu

# name -> (sites, extents, f)
LAYERS = {
    "2^3": lambda: (inputs.surfaces(2, 64, 8, 28, seed=51, target=6000), [2, 64, 64, 64], 2),
    "4^3": lambda: (inputs.surfaces(1, 32, 4, 14, seed=52, target=2000), [1, 32, 32, 32], 4),
    "8^3": lambda: (inputs.surfaces(1, 32, 4, 14, seed=53, target=2000), [1, 32, 32, 32], 8),
    "16^2": lambda: (inputs.pen_strokes(3, 64, seed=54), [3, 64, 64], 16),
    "32^2": lambda: (inputs.pen_strokes(9, 64, seed=55), [9, 64, 64], 32),
    "2^3 of 25": lambda: (_below(inputs.surfaces(2, 25, 4, 11, seed=56, target=3000), 24),
                          [2, 25, 25, 25], 2),
    "4^2 of 67": lambda: (_below(inputs.pen_strokes(4, 67, seed=57), 64), [4, 67, 67], 4),
}


def _below(c, e):
    return np.ascontiguousarray(c[(c[:, 1:] < e).all(1)])


@pytest.mark.parametrize("path", ["grid", "hash"])
@pytest.mark.parametrize("layer", list(LAYERS))
def test_reversed_layers(monkeypatch, layer, path):
    coords, size, f = LAYERS[layer]()
    coords = coords[np.random.default_rng(58).permutation(len(coords))]
    D = coords.shape[1]
    fs = [1] + [f] * (D - 1)
    monkeypatch.setenv("SPCONV_RULEBOOK", path)
    rb = spc.build_rulebook(spc.SC, _t(coords), size, fs, fs, transpose=True)
    ref = oracle.Rulebook(oracle.SC, coords, size, fs, fs)
    # every site in one pair: the pair lists, not the transposed map, are what runs
    assert int(rb.pair_off[-1]) == rb.n_in == ref.n_in
    k = np.diff(rb.pair_off)
    _say(f"[pairs] {layer} {path}: {ref.n_in} rows, {ref.n_out} fields, {ref.K} offsets of "
         f"{k.min()} to {k.max()} pairs")
    for ci, co, dtype in [(32, 64, "bf16"), (64, 16, "f32"), (24, 40, "bf16"), (5, 3, "f32"),
                          (136, 72, "f32")]:
        rtol = RTOL_F32 if dtype == "f32" else RTOL_BF16
        w = _feats(ref.K * ci, co, dtype, 1, std=1.0 / np.sqrt(ci)).reshape(ref.K, ci, co)
        b = inputs.normal_f32((co,), std=0.1, seed=2)
        x, dy = _feats(ref.n_out, ci, dtype, 3), _feats(ref.n_out, co, dtype, 4)
        y = spc.dc_forward(rb, _dev(x, dtype), _dev(w, dtype), _t(b))
        yo, ab = ref.dc_forward(x, w, b, in_dt=_odt(dtype))
        check_features(_to_np(y), yo, ab, rtol, f"DC {ci} -> {co}")
        dx = spc.backward_data(rb, spc.OP_SC, _dev(dy, dtype), _dev(w, dtype))
        dxo, ad = ref.backward_data(oracle.SC, dy, w, _odt(dtype))
        check_features(_to_np(dx), dxo, ad, rtol, f"dx {ci} -> {co}")
