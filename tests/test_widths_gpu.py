"""Channel counts around the edges of the matrix-core kernels' slabs, column
tiles and 16-byte pieces, against the oracle: forward, input gradient, weight
and bias gradients of VSC, SC and DC layers, with and without the block
epilogue, on layers of several row tiles with a remainder.  The bounds are the
ones of the other parity tests: per element rtol times the sum of absolute
terms, rtol 1e-5 for fp32, 2e-2 for bf16, 1e-4 for weight gradients."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

import oracle  # noqa: E402
import paper_1706_01307_amd as spc  # noqa: E402
from paper_1706_01307_amd import inputs  # noqa: E402
from tests import dense_ref  # noqa: E402
from tests.test_ops_gpu import OP, RTOL_GRAD, _dev, _feats, _odt  # noqa: E402
from tests.test_parity_gpu import (RTOL_BF16, RTOL_F32, _say, _t, _to_np,  # noqa: E402
                                   check_features, compare_layer)

pytestmark = pytest.mark.gpu

# one plane past and short of a slab (64 bf16, 32 fp32), of a k-chunk, of a 16-byte piece and of
# a column tile (32, 64, 96, 128 columns); rows that are no whole pieces on either or both sides
WIDTHS = [(8, 8), (24, 40), (40, 24), (72, 136), (192, 96), (136, 264), (16, 20), (31, 33),
          (65, 16), (33, 130), (5, 3), (2, 30), (48, 1), (129, 8)]


# layer -> (extent, f): overlapping fields (the transposed map), f = s on extents the stride
# divides (the pair lists) and leaves a border of, with sites there (the transposed map)
SC_LAYERS = {"map": (24, 3), "direct": (24, 2), "border": (25, 2)}


def _layer(op, layer):
    if op == "vsc":
        coords = inputs.pen_strokes(2, 64, seed=41, target=300)[:513]
        return coords, [2, 64, 64], [1, 3, 3], [1, 1, 1]
    e, f = SC_LAYERS[layer]
    return (inputs.surfaces(1, e, 4.0, 10.0, seed=42, target=700)[:700], [1] + [e] * 3,
            [1] + [f] * 3, [1, 2, 2, 2])


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("op,layer", [("vsc", "")] + [(o, k) for o in ("sc", "dc")
                                                      for k in SC_LAYERS])
@pytest.mark.parametrize("ci,co", WIDTHS + [(32, 64), (96, 32), (256, 16)])
def test_layer_and_gradients(op, layer, ci, co, dtype):
    coords, size, f, s = _layer(op, layer)
    kind = spc.VSC if op == "vsc" else spc.SC
    rb = spc.build_rulebook(kind, _t(coords), size, f, s, transpose=op != "vsc")
    ref = oracle.Rulebook(kind, coords, size, f, s)
    rin, rout = (ref.n_out, ref.n_in) if op == "dc" else (ref.n_in, ref.n_out)
    _say(f"[widths] {op} {layer} {rin} -> {rout} C={ci}->{co} {dtype}")
    x, dy = _feats(rin, ci, dtype, 1), _feats(rout, co, dtype, 2)
    wf = inputs.normal_f32((ref.K, ci, co), std=1.0 / np.sqrt(ref.K * ci), seed=3)
    w = inputs.to_bf16_bits(wf) if dtype == "bf16" else wf
    b = inputs.normal_f32((co,), std=0.1, seed=4)
    rtol = RTOL_F32 if dtype == "f32" else RTOL_BF16
    fwd = {"vsc": spc.vsc_forward, "sc": spc.sc_forward, "dc": spc.dc_forward}[op]
    y = fwd(rb, _dev(x, dtype), _dev(w, dtype), _t(b))
    yo, ab = (ref.dc_forward if op == "dc" else ref.forward)(x, w, b, in_dt=_odt(dtype))
    check_features(_to_np(y), yo, ab, rtol, "y")
    dx = spc.backward_data(rb, OP[op][0], _dev(dy, dtype), _dev(w, dtype))
    dxo, ad = ref.backward_data(OP[op][1], dy, w, _odt(dtype))
    check_features(_to_np(dx), dxo, ad, rtol, "dx")
    dw, db = spc.backward_weight(rb, OP[op][0], _dev(x, dtype), _dev(dy, dtype), ci, co)
    dwo, dbo, aw, adb = ref.backward_weight(OP[op][1], x, dy, ci, co, _odt(dtype))
    check_features(dw.cpu().numpy(), dwo, aw, RTOL_GRAD, "dw")
    check_features(db.cpu().numpy(), dbo, adb, RTOL_GRAD, "db")
    dw2, _ = spc.backward_weight(rb, OP[op][0], _dev(x, dtype), _dev(dy, dtype), ci, co)
    assert torch.equal(dw, dw2)
    if op == "vsc":
        scale = inputs.normal_f32((co,), seed=5)
        res = _feats(rout, co, dtype, 6)
        yf = spc.forward_fused(rb, _dev(x, dtype), _dev(w, dtype), scale=_t(scale), shift=_t(b),
                               residual=_dev(res, dtype), relu=True)
        y64, a64 = ref.forward(x, w, None, in_dt=_odt(dtype))
        zo, bound = oracle.fused_epilogue(y64, a64, scale, b, res, True, _odt(dtype))
        check_features(_to_np(yf), zo, bound, rtol, "fused")


@pytest.mark.parametrize("ci,co,dtype", [(40, 24, "f32"), (24, 40, "bf16"), (72, 72, "bf16"),
                                         (20, 96, "f32")])
def test_many_rows(ci, co, dtype):
    """Enough rows for the largest row tiles."""
    c = dense_ref.random_sites(np.random.default_rng(43), [1, 64, 64, 64], 0.62)
    compare_layer(spc.VSC, c, [1, 64, 64, 64], [1, 1, 1, 3], [1] * 4, ci, co, dtype=dtype,
                  what="many rows")


@pytest.mark.parametrize("ci,co,dtype", [(64, 32, "bf16"), (136, 40, "bf16"), (40, 72, "f32"),
                                         (7, 24, "f32")])
def test_many_rows_reversed(ci, co, dtype):
    """DC and the SC input gradient (f = s) on enough rows for the largest row tiles."""
    size, f = [1, 64, 64, 64], [1, 1, 1, 2]
    c = dense_ref.random_sites(np.random.default_rng(44), size, 0.62)
    c = c[np.random.default_rng(45).permutation(len(c))]
    rb = spc.build_rulebook(spc.SC, _t(c), size, f, f, transpose=True)
    ref = oracle.Rulebook(oracle.SC, c, size, f, f)
    rtol = RTOL_F32 if dtype == "f32" else RTOL_BF16
    w = _feats(2 * ci, co, dtype, 7).reshape(2, ci, co)
    b = inputs.normal_f32((co,), seed=8)
    x, dy = _feats(ref.n_out, ci, dtype, 9), _feats(ref.n_out, co, dtype, 10)
    y = spc.dc_forward(rb, _dev(x, dtype), _dev(w, dtype), _t(b))
    yo, ab = ref.dc_forward(x, w, b, in_dt=_odt(dtype))
    check_features(_to_np(y), yo, ab, rtol, "DC")
    dx = spc.backward_data(rb, spc.OP_SC, _dev(dy, dtype), _dev(w, dtype))
    dxo, ad = ref.backward_data(oracle.SC, dy, w, _odt(dtype))
    check_features(_to_np(dx), dxo, ad, rtol, "dx")


@pytest.mark.parametrize("path", ["slab", "vec"])
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("op,layer", [("vsc", ""), ("sc", "map"), ("dc", "map")])
@pytest.mark.parametrize("ci,co", [(8, 8), (24, 40), (31, 33), (65, 16), (5, 3), (48, 1),
                                   (12, 100), (129, 8)])
def test_either_kernel(monkeypatch, op, layer, ci, co, dtype, path):
    """The matrix cores' slabs and one lane per column, whichever of them the dispatch takes for
    these layers: forward and input gradient."""
    monkeypatch.setenv("SPCONV_FORCE_PATH", path)
    coords, size, f, s = _layer(op, layer)
    kind = spc.VSC if op == "vsc" else spc.SC
    rb = spc.build_rulebook(kind, _t(coords), size, f, s, transpose=op != "vsc")
    ref = oracle.Rulebook(kind, coords, size, f, s)
    rin, rout = (ref.n_out, ref.n_in) if op == "dc" else (ref.n_in, ref.n_out)
    x, dy = _feats(rin, ci, dtype, 1), _feats(rout, co, dtype, 2)
    w = _feats(ref.K * ci, co, dtype, 3, std=1.0 / np.sqrt(ref.K * ci)).reshape(ref.K, ci, co)
    b = inputs.normal_f32((co,), std=0.1, seed=4)
    rtol = RTOL_F32 if dtype == "f32" else RTOL_BF16
    fwd = {"vsc": spc.vsc_forward, "sc": spc.sc_forward, "dc": spc.dc_forward}[op]
    yo, ab = (ref.dc_forward if op == "dc" else ref.forward)(x, w, b, in_dt=_odt(dtype))
    check_features(_to_np(fwd(rb, _dev(x, dtype), _dev(w, dtype), _t(b))), yo, ab, rtol, "y")
    dxo, ad = ref.backward_data(OP[op][1], dy, w, _odt(dtype))
    dx = spc.backward_data(rb, OP[op][0], _dev(dy, dtype), _dev(w, dtype))
    check_features(_to_np(dx), dxo, ad, rtol, "dx")


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_reversed_on_the_vector_path(monkeypatch, dtype):
    """The f = s reversed direction without the matrix cores gives the same results within the
    two paths' bounds."""
    coords, size, f, s = _layer("dc", "direct")
    rb = spc.build_rulebook(spc.SC, _t(coords), size, f, s, transpose=True)
    ref = oracle.Rulebook(oracle.SC, coords, size, f, s)
    x, w = _feats(ref.n_out, 20, dtype, 1), _feats(8 * 20, 12, dtype, 2).reshape(8, 20, 12)
    monkeypatch.setenv("SPCONV_FORCE_PATH", "vec")
    y = spc.dc_forward(rb, _dev(x, dtype), _dev(w, dtype))
    yo, ab = ref.dc_forward(x, w, None, in_dt=_odt(dtype))
    check_features(_to_np(y), yo, ab, RTOL_F32 if dtype == "f32" else RTOL_BF16, "DC")
    g = _feats(ref.n_out, 12, dtype, 3)
    dx = spc.backward_data(rb, spc.OP_SC, _dev(g, dtype), _dev(w, dtype))
    dxo, ad = ref.backward_data(oracle.SC, g, w, _odt(dtype))
    check_features(_to_np(dx), dxo, ad, RTOL_F32 if dtype == "f32" else RTOL_BF16, "dx")


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("op,layer,ci,co", [("vsc", "", 24, 40), ("vsc", "", 33, 130),
                                            ("vsc", "", 200, 72), ("sc", "map", 136, 24),
                                            ("dc", "map", 40, 24), ("dc", "direct", 40, 24)])
def test_nonfinite_weights_stay_with_their_pairs(op, layer, ci, co, dtype):
    """An infinity and a NaN in W^i reach the rows that have a neighbour at offset i and no other,
    as the sum over the pairs says: forward, input gradient and the in-place fused forward."""
    coords, size, f, s = _layer(op, layer)
    kind = spc.VSC if op == "vsc" else spc.SC
    rb = spc.build_rulebook(kind, _t(coords), size, f, s, transpose=op != "vsc")
    ref = oracle.Rulebook(kind, coords, size, f, s)
    rin, rout = (ref.n_out, ref.n_in) if op == "dc" else (ref.n_in, ref.n_out)
    x, dy = _feats(rin, ci, dtype, 1), _feats(rout, co, dtype, 2)
    w = _feats(ref.K * ci, co, dtype, 3, std=1.0 / np.sqrt(ref.K * ci)).reshape(ref.K, ci, co)
    inf, nan = (0x7f80, 0x7fc0) if dtype == "bf16" else (np.inf, np.nan)
    w[1, 3, 2], w[ref.K - 2, ci - 1, co - 1] = inf, nan
    b = inputs.normal_f32((co,), std=0.1, seed=4)
    rtol = RTOL_F32 if dtype == "f32" else RTOL_BF16

    def check(got, want, bound, what):
        got = _to_np(got).astype(np.float64)
        ok = np.isfinite(want)
        assert not ok.all() and ok.any(), what
        np.testing.assert_array_equal(got[~ok], want[~ok], err_msg=what)     # NaN where NaN
        assert (np.abs(got - want)[ok] <= rtol * bound[ok]).all(), what

    with np.errstate(invalid="ignore"):
        fwd = {"vsc": spc.vsc_forward, "sc": spc.sc_forward, "dc": spc.dc_forward}[op]
        yo, ab = (ref.dc_forward if op == "dc" else ref.forward)(x, w, b, in_dt=_odt(dtype))
        check(fwd(rb, _dev(x, dtype), _dev(w, dtype), _t(b)), yo, ab, "y")
        dxo, ad = ref.backward_data(OP[op][1], dy, w, _odt(dtype))
        check(spc.backward_data(rb, OP[op][0], _dev(dy, dtype), _dev(w, dtype)), dxo, ad, "dx")
        if op != "dc":
            scale, res = inputs.normal_f32((co,), seed=5), _feats(rout, co, dtype, 6)
            y64, a64 = ref.forward(x, w, None, in_dt=_odt(dtype))
            zo, bound = oracle.fused_epilogue(y64, a64, scale, b, res, True, _odt(dtype))
            z = _dev(res, dtype)
            spc.forward_fused(rb, _dev(x, dtype), _dev(w, dtype), scale=_t(scale), shift=_t(b),
                              residual=z, relu=True, out=z)
            check(z, zo, bound, "fused")


@pytest.mark.parametrize("op", ["vsc", "dc"])
def test_more_columns_than_a_grid_has_tiles(op):
    """4,194,308 output planes: one past 65535 tiles of 64 columns."""
    co = 65535 * 64 + 68
    c = np.array([[0, 1, 2], [0, 1, 3], [0, 5, 5]], np.int32)
    rb = spc.build_rulebook(spc.VSC if op == "vsc" else spc.SC, _t(c), [1, 8, 8], [1, 1, 1],
                            transpose=op == "dc")
    g = torch.Generator("cuda").manual_seed(1)
    x = torch.randn(3, 5, device="cuda", generator=g)
    w = torch.randn(1, 5, co, device="cuda", generator=g)
    y = (spc.vsc_forward if op == "vsc" else spc.dc_forward)(rb, x, w)
    want, bound = x.double() @ w[0].double(), x.double().abs() @ w[0].double().abs()
    assert ((y.double() - want).abs() <= RTOL_F32 * bound).all()


@pytest.mark.parametrize("size,f,s", [([3, 101, 77, 95], [1, 3, 3, 3], [1, 2, 2, 2]),
                                      ([2, 130, 100, 90], [1, 2, 2, 2], [1, 2, 2, 2]),
                                      ([1, 300, 1000], [1, 1, 2], [1, 1, 1]),
                                      ([1, 1100, 1100], [1, 3, 1], [1, 2, 1])])
def test_strided_book_on_large_output_grids(size, f, s):
    """Output grids past 2^18 cells with at most 64 cells per input site (marked byte by byte),
    and one with more (marked by bits)."""
    n = 3000 if size[1] == 1100 else 30000
    rng = np.random.default_rng(46)
    c = np.unique(np.stack([rng.integers(0, e, n) for e in size], 1), axis=0).astype(np.int32)
    compare_layer(spc.SC, c[rng.permutation(len(c))], size, f, s, 16, 16, what="large outputs")
