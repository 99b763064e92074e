"""Edge sizes of the kernels' tiles, remainders and dispatch lines, against the CPU oracle (bars as in test_gpu_kan)."""
import ctypes

import numpy as np
import pytest
import torch

import oracle
from paper_2408_11200_amd import binding, workloads
from test_gpu_kan import GRAD_TOL, assert_close, dev, run_layer_parity
from test_gpu_ukan import make as ukan_make, run as ukan_run

pytestmark = pytest.mark.gpu


def families_of(call):
    """The kernel families that a call launches."""
    seen = set()
    hook = ctypes.CFUNCTYPE(None, ctypes.c_char_p, ctypes.c_void_p)(lambda family, stream: seen.add(family.decode()))
    none = ctypes.CFUNCTYPE(None, ctypes.c_char_p, ctypes.c_void_p)(lambda family, stream: None)
    binding.kan_set_launch_observer(hook, none)
    try:
        call()
    finally:
        binding.kan_set_launch_observer(None, None)
    torch.cuda.synchronize()
    return seen


def run_with_families(w):
    """Parity of a layer's backward pass; returns the kernel families that it launched."""
    s, p = w.layers[0], w.params[0]
    run_layer_parity(w, gx_in_grid_units=s.G > 1000)
    x, coef, w_s, w_b, gy = (dev(a) for a in (w.x, p["coef"], p["w_s"], p["w_b"], w.gy))
    return families_of(lambda: binding.kan_backward(s, x, coef, w_s, w_b, gy))


def forward_with_families(w):
    """Parity of a layer's forward pass; returns the kernel families that it launched."""
    s, p = w.layers[0], w.params[0]
    run_layer_parity(w, check_grads=False)
    x, coef, w_s, w_b = (dev(a) for a in (w.x, p["coef"], p["w_s"], p["w_b"]))
    return families_of(lambda: binding.kan_forward(s, x, coef, w_s, w_b))


@pytest.mark.parametrize("B,n_in,n_out,G,k", [
    (1, 1, 1, 1, 1),                   # one pair
    (5, 31, 16, 3, 3),                 # four waves, exactly one 16-lane tile
    (3, 33, 17, 10, 2),                # sixteen waves, ragged 32-lane tile
    (2, 1100, 33, 4, 3),               # more inputs than one round of pair evaluations, ragged 64-lane tile
    (2049, 40, 65, 6, 3),              # four samples per workgroup, ragged batch, the last lane moved back
    (2050, 600, 5, 6, 3),              # narrowest tile of four outputs per lane, running sums folded
    (2048, 3, 3, 6, 3),                # fewer outputs than a lane takes
    (4099, 35, 30, 40, 3), (2050, 35, 126, 6, 1),
    (9, 70, 130, 12, 5), (2047, 20, 64, 5, 4), (5001, 20, 31, 5, 5),      # window of six rows
    (16384, 5, 64, 8, 3), (16385, 5, 64, 8, 3),     # the last batch of the direct kernel and the first past it
])
def test_small_batch_forward(B, n_in, n_out, G, k):
    w = workloads.random_kan_layer(B + n_in, B, n_in, n_out, G, k, outside_frac=0.2)
    y, _ = run_layer_parity(w, check_grads=False)
    s, p = w.layers[0], w.params[0]
    x, coef, w_s, w_b, gy = (dev(a) for a in (w.x, p["coef"], p["w_s"], p["w_b"], w.gy))
    # the entry point that keeps no table gives the same sums, and the one that does leaves it behind
    assert torch.equal(y, binding.kan_forward_static(s, x, coef, w_s, w_b, torch.empty_like(y)))
    ws = torch.empty(binding.kan_workspace_bytes(s, B), dtype=torch.uint8, device="cuda")
    binding.kan_forward(s, x, coef, w_s, w_b, ws=ws)
    table = torch.cat([coef * w_s[:, None, :], w_b[:, None, :]], dim=1)
    assert torch.equal(ws[:table.numel() * 4].view(torch.float32), table.flatten())


@pytest.mark.parametrize("k", [3, 5])
@pytest.mark.parametrize("n_out", [65, 66, 67, 129, 130, 131, 193, 195])
def test_tile_whose_lane_starts_in_the_tile_before(n_out, k):
    """One to three outputs past a tile of 64 at four outputs per lane: the last lane's outputs begin in the tile before."""
    run_layer_parity(workloads.random_kan_layer(n_out, 2051, 9, n_out, 7, k, outside_frac=0.1), check_grads=False)


@pytest.mark.parametrize("B,n_in,n_out,G,k", [
    (33000, 8, 17, 18000, 3), (40000, 9, 18, 20000, 1),     # two outputs a lane, tables past L2, ragged rows
    (66000, 17, 31, 5000, 2), (66005, 8, 32, 3000, 3),      # tables in L2, an input past sixteen; a whole tile
    (33000, 17, 30, 6000, 5),                               # two a lane, window of six rows
    (16400, 17, 33, 5000, 3), (16403, 9, 64, 9000, 3), (66000, 16, 33, 9, 4),       # four a lane
])
def test_row_stream_kernel(B, n_in, n_out, G, k):
    assert "forward_rows" in forward_with_families(workloads.random_kan_layer(n_in, B, n_in, n_out, G, k, outside_frac=0.1))


@pytest.mark.parametrize("B,n_in,n_out,G,k,family", [
    (8192, 7, 17, 6, 3, "direct"), (8193, 7, 17, 6, 3, "generic"),      # few inputs: the line and past it
    (4097, 2, 3, 6, 3, "narrow"), (4100, 3, 130, 6, 3, "lds"), (16500, 7, 62, 30, 5, "generic"),
    (2048, 8, 1, 7, 3, "direct"), (2049, 8, 2, 7, 4, "generic"),        # one to three outputs
    (2051, 8, 1, 7, 3, "direct"), (8193, 64, 2, 7, 3, "narrow"),
    (65540, 34, 9, 20, 3, "narrow"), (66000, 33, 31, 9, 1, "direct"), (33000, 8, 17, 6, 3, "direct"),
    (16400, 33, 64, 40, 3, "lds_rows"), (33000, 17, 30, 2500, 5, "direct"),
    (300, 16, 40, 1700, 3, "direct"), (300, 16, 40, 1500, 2, "direct"),         # folds of just more and less than 2^20 floats
])
def test_forward_lines(B, n_in, n_out, G, k, family):
    w = workloads.random_kan_layer(n_in, B, n_in, n_out, G, k, outside_frac=0.1)
    assert "forward_" + family in forward_with_families(w)


@pytest.mark.parametrize("B,n_in,n_out,G,k,family", [
    (34443, 32, 32, 131, 4, "direct"), (40000, 32, 32, 131, 4, "lds_rows"),     # a round of workgroups full enough
    (66594, 32, 32, 200, 5, "direct"),                                          # a second round of five
    (19738, 14, 32, 324, 5, "direct"), (23000, 14, 32, 324, 5, "lds_rows"),
    (12493, 13, 59, 85, 5, "direct"), (14800, 13, 59, 85, 5, "lds_rows"),
    (9649, 12, 40, 30, 4, "direct"), (12000, 12, 40, 30, 4, "lds_rows"),
])
def test_forward_lines_of_six_rows(B, n_in, n_out, G, k, family):
    assert "forward_" + family in forward_with_families(workloads.random_kan_layer(n_in, B, n_in, n_out, G, k))


@pytest.mark.parametrize("B,n_in,n_out,G,k", [
    (16400, 33, 64, 40, 3), (16403, 37, 35, 17, 1),             # eight waves: steps of four inputs, the last one of one
    (20000, 34, 63, 100, 3), (33000, 9, 32, 240, 3),            # steps of two; tiles of 32
    (65500, 11, 64, 10, 3), (131000, 3, 32, 256, 3),            # sixteen waves: steps of four inputs, of one
    (66000, 35, 33, 40, 2), (70001, 5, 64, 150, 3), (70000, 66, 47, 240, 3),    # eight samples a group: one to four copies a thread
    (131100, 4, 32, 60, 3), (131072 + 512, 7, 32, 100, 3), (131073, 34, 32, 300, 3),       # the same on tiles of 32, x by fours
    (45000, 9, 70, 300, 3),                                     # three tiles, the last of six outputs
    (8190, 21, 255, 200, 3), (16300, 17, 67, 50, 2), (8192, 19, 256, 245, 5),       # eight waves on several tiles
    (16400, 33, 64, 40, 5), (20000, 37, 35, 17, 4), (40000, 9, 32, 240, 5),     # windows of six rows: eight waves,
    (65500, 18, 64, 10, 5), (45000, 9, 70, 300, 4),             # sixteen,
    (66000, 35, 50, 40, 4), (131100, 9, 32, 60, 5),             # eight samples a group
])
@pytest.mark.parametrize("outside", [0.0, 0.1])
def test_lds_rows_kernel(B, n_in, n_out, G, k, outside):
    assert "forward_lds_rows" in forward_with_families(workloads.random_kan_layer(n_in, B, n_in, n_out, G, k, outside_frac=outside))


@pytest.mark.parametrize("B,n_in,n_out,G,k", [
    (16448, 33, 64, 40, 3), (20032, 37, 35, 17, 1), (33024, 9, 32, 240, 3),     # eight waves, tiles of 64 and 32
    (65536, 11, 64, 10, 3), (131072, 3, 32, 256, 3),                            # sixteen, four samples a group
    (65600, 11, 64, 10, 3), (131072, 35, 64, 40, 2), (131136, 34, 32, 300, 3),  # eight samples
    (16448, 33, 64, 40, 5), (33024, 9, 32, 60, 4), (65536, 18, 64, 10, 5), (66048, 35, 50, 40, 4), (131136, 9, 32, 60, 5),
])
def test_lds_rows_waves_in_either_order_give_the_same_bits(B, n_in, n_out, G, k):
    """A wave evaluates its pairs before the multiply-adds of a step or behind them, of windows of six rows half a workgroup's waves
    each: the same 64 samples over and over, so in every wave, have to give the same bits, inputs of several rounds included."""
    w = workloads.random_kan_layer(n_in, 64, n_in, n_out, G, k, outside_frac=0.1)
    s, p = w.layers[0], w.params[0]
    x, coef, w_s, w_b = (dev(a) for a in (w.x, p["coef"], p["w_s"], p["w_b"]))
    x = x.repeat(B // 64, 1)
    out = []
    assert "forward_lds_rows" in families_of(lambda: out.append(binding.kan_forward(s, x, coef, w_s, w_b)))
    assert torch.equal(out[0], out[0][:64].repeat(B // 64, 1))


def test_batch_past_the_threads_of_one_launch():
    """64 threads a sample: 2^26 samples are more than one launch takes.  Both ends and the seam between the parts agree
    with a call on those rows alone."""
    B, n_out = (1 << 26) + 5, 17
    w = workloads.random_kan_layer(3, 16, 1, n_out, 6, 3)
    s, p = w.layers[0], w.params[0]
    coef, w_s, w_b = (dev(p[n]) for n in ("coef", "w_s", "w_b"))
    x = torch.rand((B, 1), device="cuda") * 2 - 1
    y = binding.kan_forward(s, x, coef, w_s, w_b)
    for lo in (0, (1 << 25) - 2050, B - 4100):
        part = x[lo:lo + 4100].clone()
        assert torch.equal(y[lo:lo + 4100], binding.kan_forward(s, part, coef, w_s, w_b)), lo


@pytest.mark.parametrize("B,n_in,n_out,G,k", [
    (700, 5, 17, 9, 3), (1100, 4, 33, 9, 3), (900, 4, 63, 12, 2),   # dense basis rows
    (700, 5, 31, 300, 3),                           # generic: few samples, few inputs, a long table
    (900, 3, 65, 9, 3), (2100, 3, 127, 40, 1),      # two streams
    (900, 3, 130, 9, 3), (700, 3, 255, 10, 3),      # one stream
    (600, 2, 257, 9, 3), (600, 2, 300, 9, 3), (500, 2, 515, 9, 3),      # one stream, two tiles and three
    (700, 4, 35, 10, 5),                            # two records per pair
])
def test_widths_that_are_no_multiple_of_the_lanes(B, n_in, n_out, G, k):
    run_layer_parity(workloads.random_kan_layer(n_out, B, n_in, n_out, G, k, outside_frac=0.2))


@pytest.mark.parametrize("B,n_in,n_out,G,k,family", [
    (256, 7, 37, 100, 3, "dparam_generic"), (257, 7, 37, 100, 3, "backward_walk"),
    (128, 2, 127, 100, 3, "dparam_generic"), (129, 2, 127, 100, 3, "backward_walk"),
    (512, 31, 19, 2000, 2, "dparam_generic"), (512, 32, 19, 2000, 2, "backward_walk"),
    (64, 8, 63, 80, 5, "dparam_generic"), (64, 8, 64, 80, 5, "backward_walk"),
    (64, 3, 193, 70, 3, "backward_walk"), (64, 3, 20, 70, 3, "backward_walk"),
])
def test_few_samples_of_ragged_widths(B, n_in, n_out, G, k, family):
    assert family in run_with_families(workloads.random_kan_layer(n_out, B, n_in, n_out, G, k, outside_frac=0.1))


@pytest.mark.parametrize("B,n_in,n_out,G,k", [
    (1500, 33, 31, 100, 3),            # two outputs per lane, the last lane moved back: single-level sums,
    (20000, 14, 17, 80, 3),            # two-level sums of chunks of 2048,
    (3000, 40, 19, 1100, 3),           # zeroed tables that the walk jumps through
    (9000, 9, 37, 70, 3), (9000, 9, 63, 90, 1),     # four per lane, many segments
    (70000, 8, 18, 9, 3),              # two per lane, many segments of few rows
    (900, 40, 47, 2000, 3),            # four per lane, zeroed tables
])
def test_ragged_walk(B, n_in, n_out, G, k):
    assert "backward_walk" in run_with_families(workloads.random_kan_layer(n_out + 5, B, n_in, n_out, G, k, outside_frac=0.1))


@pytest.mark.parametrize("B,n_in,n_out,G,k", [
    (8200, 16, 257, 9, 3), (8200, 17, 509, 5, 2), (8200, 16, 777, 5, 3),        # eight outputs per lane, ragged: one tile and two
    (8191, 16, 257, 9, 3), (8200, 16, 256 + 512, 6, 3), (8200, 15, 301, 9, 3),  # just not; a multiple of eight; too few inputs
    (14500, 4, 264, 40000, 3),                      # partial sums ask for chunks of 2048: four outputs per lane
    (4200, 16, 385, 9, 5),
])
def test_walk_of_wide_layers(B, n_in, n_out, G, k):
    assert "backward_walk" in run_with_families(workloads.random_kan_layer(n_out, B, n_in, n_out, G, k, outside_frac=0.05))


@pytest.mark.parametrize("B,n_in,n_out,G,k", [
    (32800, 7, 30, 20, 3), (16400, 5, 37, 20, 3),                   # generic; long-table kernel
    (16400, 70, 63, 700, 3),                                        # row-stream kernel
    (16400, 40, 9, 20, 3), (65540, 34, 9, 20, 3),                   # direct, and the narrow kernel past it
    (8200, 20, 127, 600, 3), (4200, 10, 260, 400, 3),               # direct after the fold kernel, generic
    (11000, 9, 130, 15, 3), (5200, 5, 259, 15, 3),                  # LDS-staged kernels
    (16400, 8, 50, 700, 5), (7300, 4, 131, 12, 4),                  # window of six rows: direct, LDS-staged
])
def test_large_batches_of_ragged_widths(B, n_in, n_out, G, k):
    run_layer_parity(workloads.random_kan_layer(n_out + 1, B, n_in, n_out, G, k, outside_frac=0.1))


def test_ragged_width_on_shared_partial_tables():
    """Several rounds of chunks on one partial table: outputs two lanes share are added once."""
    run_layer_parity(workloads.random_kan_layer(5, 220000, 3, 35, 400000, 3, outside_frac=0.0), gx_in_grid_units=True)


@pytest.mark.parametrize("B,n_in,n_out,G,k", [
    (8192, 2, 3, 5, 3), (9000, 3, 4, 700, 3),       # one output per lane; row slices added by a second kernel
    (70000, 2, 18, 9, 3),                           # dense basis rows: many chunks
    (33000, 3, 34, 3, 2),                           # many segments of few rows, ragged tiles
    (2500, 40, 520, 6, 3),                          # small workgroups (more than 512 of them), two tiles
    (40000, 3, 20, 1030, 5),                        # two records per pair, long table
])
def test_reduction_over_the_chunks(B, n_in, n_out, G, k):
    run_layer_parity(workloads.random_kan_layer(n_out + 7, B, n_in, n_out, G, k, outside_frac=0.1))


@pytest.mark.parametrize("B,n_in,n_out,G,k", [
    (300000, 1, 33, 10, 3),                         # more segments than are kept in LDS, many to a row
    (66000, 2, 1, 140000, 3), (66000, 2, 2, 9000, 3), (33000, 3, 3, 300, 3),    # one, two, three outputs; rows share a mark
    (33000, 5, 20, 64, 3), (33000, 5, 20, 61, 3),   # 67 rows: the first table in slices; 64: the last that is not
    (3000, 300, 40, 200, 3),                        # slices of more than the smallest number of rows
])
def test_reduction_adds_the_carry_rows(B, n_in, n_out, G, k):
    assert run_with_families(workloads.random_kan_layer(n_out + 9, B, n_in, n_out, G, k, outside_frac=0.05)) >= {"backward_walk", "dparam_reduce"}


@pytest.mark.parametrize("B,n_in,n_out,G,k", [
    (1, 2, 1, 1, 1), (255, 3, 5, 12, 3), (257, 2, 16, 12, 3),       # one tile of 16 rows (12 + 3 + the base row) and outputs
    (1000, 2, 17, 13, 3), (700, 3, 32, 28, 3),                      # just past a tile; the last of two tiles
    (600, 2, 33, 29, 3), (513, 2, 64, 60, 3), (513, 2, 64, 61, 3),  # four tiles; the first length left to the walk
    (65536, 16, 5, 9, 2), (65537, 16, 5, 9, 2),                     # eight sub-chunks a chunk; the first batch left to the walk
])
def test_dense_basis_backward(B, n_in, n_out, G, k):
    run_layer_parity(workloads.random_kan_layer(n_out + 11, B, n_in, n_out, G, k, outside_frac=0.2))


def test_dense_basis_backward_keeps_a_non_finite_gradient_to_its_rows():
    w = workloads.random_kan_layer(3, 500, 2, 5, 10, 3, outside_frac=0.1)
    s, p = w.layers[0], w.params[0]
    x, coef, w_s, w_b, gy = (dev(a) for a in (w.x, p["coef"], p["w_s"], p["w_b"], w.gy))
    bad = gy.clone()
    bad[300, 2] = float("inf")
    good, got = (binding.kan_backward(s, x, coef, w_s, w_b, t) for t in (gy, bad))
    idx = binding.kan_interval_index(s, x)[300].tolist()
    for i, cell in enumerate(idx):
        for m in range(s.G + s.k):
            touched = cell <= m <= cell + s.k
            assert bool(torch.isfinite(got["gcoef"][i, m, 2])) == (not touched), (i, m, cell)
    keep = [0, 1, 3, 4]
    assert torch.allclose(got["gcoef"][:, :, keep], good["gcoef"][:, :, keep], rtol=1e-5, atol=1e-6)


@pytest.mark.parametrize("where", ["gy", "coef"])
def test_dense_basis_backward_multiplies_a_zero_weight(where):
    """On a knot the last weight of the window and its derivative are zero, and so is SiLU at zero: times an infinite
    gradient or coefficient they are NaN, not left out."""
    w = workloads.random_kan_layer(4, 500, 2, 5, 10, 3, outside_frac=0.1)
    w.x[300] = 0.0
    s, p = w.layers[0], w.params[0]
    if where == "gy":
        w.gy[300, 2] = np.inf
    else:
        p["coef"][:, 8, 2] = np.inf
    x, coef, w_s, w_b, gy = (dev(a) for a in (w.x, p["coef"], p["w_s"], p["w_b"], w.gy))
    got = {n: t.cpu().numpy() for n, t in binding.kan_backward(s, x, coef, w_s, w_b, gy).items()}
    with np.errstate(invalid="ignore"):
        ref = oracle.kan_backward(w.x, p["coef"], p["w_s"], p["w_b"], w.gy, s.G, s.k, s.grid_lo, oracle.inv_h_of(s.grid_lo, s.grid_hi, s.G))
    assert not np.isfinite(ref["gx"][300]).any()
    for name in ("gx", "gcoef", "gw_b"):
        np.testing.assert_array_equal(np.isfinite(got[name]), np.isfinite(ref[name]), name)
    if where == "gy":
        assert np.isnan(ref["gcoef"][:, 8, 2]).all() and np.isnan(ref["gw_b"][:, 2]).all()


@pytest.mark.parametrize("B,n_in,n_out,kw", [
    (257, 260, 2, dict()),                                   # four inputs a lane, two input tiles, a second strip of one row
    (300, 259, 3, dict()),                                   # one input a lane, five tiles
    (40000, 3, 1, dict(xs=1.0)),                             # every strip of the range scan
    (60, 2, 3, dict(d_pe=34, d_feat=31, d_hid=65)),          # rows and columns past the tiles of the generator kernels
    (40, 2, 2, dict(d_pe=130, d_feat=130, d_hid=70)),        # first generator weights too large for LDS
    (20, 1, 2, dict(d_pe=800, d_feat=400, d_hid=5)),         # one generator row a workgroup
    (2000, 4, 20, dict(base_act=1, xs=1.0)),                 # dense-basis backward on a generated table
    (5000, 3, 40, dict(k=4, xs=1.0)),
])
def test_ukan_generator_and_range_edges(B, n_in, n_out, kw):
    spec, p, x, gy = ukan_make(B + n_in, B, n_in, n_out, **kw)
    ukan_run(spec, p, x, np.float32(gy / np.sqrt(B)))


@pytest.mark.parametrize("d_hid,d_feat", [(512, 300), (513, 300), (2100, 8), (5200, 8)])
def test_ukan_wide_hidden_layers(d_hid, d_feat):
    """Embedding gradients: one tile of hidden columns and more, for more features than a workgroup has threads."""
    spec, p, x, gy = ukan_make(d_hid, 30, 2, 2, d_hid=d_hid, d_feat=d_feat)
    ukan_run(spec, p, x, np.float32(gy / np.sqrt(30)))


def test_ukan_generator_rows_past_one_dimension_of_a_launch():
    """Wide encodings take a generator row a workgroup; 65535 inputs of 257 groups are more rows than one dimension holds.
    The layer is the sum of the layers over each half of its inputs."""
    n_in, cut = 65535, 32768
    spec, p, x, _ = ukan_make(9, 2, n_in, 1, d_pe=1000, d_feat=4, d_hid=1)
    x[0], x[1] = -32.0 + np.float32(1e-3), 223.5           # 256 groups of width one, and the one before them
    P = {n: dev(a) for n, a in p.items()}
    y = binding.ukan_cg_forward(spec, dev(x), P, 257)
    parts = []
    for sl in (slice(0, cut), slice(cut, n_in)):
        half = workloads.UkanLayerSpec(sl.stop - sl.start, 1, spec.k, spec.h, spec.d_pe, spec.d_feat, spec.d_hidden, 0)
        Q = {n: (t[sl].clone() if n in ("E", "scale") else t) for n, t in P.items()}
        parts.append(binding.ukan_cg_forward(half, dev(x[:, sl]), Q, 257).double())
    total = parts[0] + parts[1]
    # fp32 sums of 65535 terms, folded every 32: a few units in the last place of the largest part
    bound = 1e-5 * float(parts[0].abs().max() + parts[1].abs().max() + 1.0)
    assert float((y.double() - total).abs().max()) <= bound


@pytest.mark.parametrize("B,n_in,n_out,kw", [
    (40, 1, 1, dict(d_hid=1)), (300, 40, 17, dict(d_hid=65, xs=10.0)),      # one column; several slices, ragged steps and columns
])
def test_ukan_bias_gradients_alone_in_slices(B, n_in, n_out, kw):
    """Both bias gradients, each without its weights' gradient, are those of the full pass bit for bit."""
    spec, p, x, gy = ukan_make(B, B, n_in, n_out, **kw)
    pd = {n: dev(a) for n, a in p.items()}
    every = binding.ukan_cg_backward(spec, dev(x), pd, dev(gy), 160)
    some = binding.ukan_cg_backward(spec, dev(x), pd, dev(gy), 160, want=("gb1", "gb2"))
    assert torch.equal(some["gb1"], every["gb1"]) and torch.equal(some["gb2"], every["gb2"])


@pytest.mark.parametrize("want", [("gb2",), ("gW2",), ("gb1",), ("gW1", "gE")])
def test_ukan_bias_gradients_alone(want):
    spec, p, x, gy = ukan_make(5, 400, 3, 33)
    pd = {n: dev(a) for n, a in p.items()}
    every = binding.ukan_cg_backward(spec, dev(x), pd, dev(gy), 64)
    some = binding.ukan_cg_backward(spec, dev(x), pd, dev(gy), 64, want=want)
    assert set(some) == set(want)
    for n in want:
        assert torch.equal(some[n], every[n]), n


@pytest.mark.parametrize("B,n_in,n_out,G,k", [
    (66000, 8, 2, 1022, 2), (66000, 8, 2, 1025, 3),        # lists of 8192 keys: the last table of one pass, the first of two
    (33000, 16, 66, 2047, 1), (33000, 16, 66, 2050, 1),    # lists of 4096, 11-bit digits
    (1030, 70, 20, 70, 3), (2500, 5, 20, 2200, 3),         # lists of 256 keys
    (9000, 8, 20, 2100, 4),                                # two records per pair
])
def test_sort_passes(B, n_in, n_out, G, k):
    run_layer_parity(workloads.random_kan_layer(G, B, n_in, n_out, G, k, outside_frac=0.05), gx_in_grid_units=True)


@pytest.mark.parametrize("B,n_in,n_out,G,k,family", [
    (1000, 4, 64, 256, 3, "walk_cells"), (1000, 4, 64, 257, 3, "walk_sort"),      # a sample a cell, and less
    (1000, 4, 256, 128, 3, "walk_cells"), (1000, 4, 256, 129, 3, "walk_sort"),    # two at one stream a wave
    (1000, 4, 128, 86, 4, "walk_cells"), (1000, 4, 128, 87, 4, "walk_sort"),      # three with two streams and six rows
    (8192, 8, 20, 1024, 3, "walk_cells"), (8192, 8, 20, 1025, 3, "walk_sort"),    # the longest table one counting pass sorts
    (255, 1, 1, 70, 1, "walk_cells"), (4097, 9, 13, 70, 2, "walk_cells"),         # one output a lane
    (2100, 33, 300, 30, 3, "walk_cells"), (9000, 67, 515, 7, 3, "walk_cells"),    # eight outputs a lane; a ragged last tile
    (16600, 16, 260, 7, 3, "walk_cells"), (16385, 40, 510, 21, 2, "walk_cells"),  # chunks of 1024 for the balance of the XCDs
    (20000, 70, 33, 30, 3, "walk_cells"),                                         # sums in two levels
    (5000, 40, 130, 30, 5, "walk_cells"), (5000, 9, 20, 64, 5, "walk_cells"), (700, 3, 96, 12, 4, "walk_cells"),
])
def test_walk_over_padded_cells(B, n_in, n_out, G, k, family):
    """Backward pass over cell lists padded to quads, either side of the lines to the record lists."""
    assert family in run_with_families(workloads.random_kan_layer(B + n_out, B, n_in, n_out, G, k, outside_frac=0.1))


@pytest.mark.parametrize("B,n_in,n_out,G", [(700, 3, 256, 40), (700, 3, 600, 30), (700, 3, 100, 40), (700, 3, 20, 70)])
def test_walk_over_padded_cells_keeps_infinities_apart(B, n_in, n_out, G):
    """An infinite and a NaN gradient reach their samples' dL/dx and the rows under their windows, and nothing else: the pads
    beside them read zeros."""
    w = workloads.random_kan_layer(n_out, B, n_in, n_out, G, 3)
    s, p = w.layers[0], w.params[0]
    x, coef, w_s, w_b, gy = (dev(a) for a in (w.x, p["coef"], p["w_s"], p["w_b"], w.gy))
    gy[[5, 300]] = 0.0
    clean = binding.kan_backward(s, x, coef, w_s, w_b, gy)
    gy[5, 1], gy[300, n_out - 1] = float("inf"), float("nan")
    g = binding.kan_backward(s, x, coef, w_s, w_b, gy)
    rest = torch.ones(B, dtype=torch.bool, device="cuda")
    rest[[5, 300]] = False
    assert torch.equal(g["gx"][rest], clean["gx"][rest]) and not torch.isfinite(g["gx"][~rest]).any()
    cell = binding.kan_interval_index(s, x).clamp(0, s.G - 1)
    for i in range(n_in):
        touched = torch.zeros((s.G + s.k, n_out), dtype=torch.bool, device="cuda")
        for b, j in ((5, 1), (300, n_out - 1)):
            touched[cell[b, i]:cell[b, i] + 4, j] = True
        assert torch.equal(g["gcoef"][i][~touched], clean["gcoef"][i][~touched])
        assert not torch.isfinite(g["gcoef"][i][touched]).any()


@pytest.mark.parametrize("B,n_in,n_out,G,k", [
    (256, 3, 256, 14, 3), (2430, 66, 260, 14, 3), (2313, 58, 384, 13, 2), (1900, 32, 515, 56, 4), (300, 2, 100, 30, 5), (300, 5, 40, 70, 3),
    (1111, 9, 20, 70, 3), (700, 7, 13, 70, 2),
])
def test_quads_past_a_batch(B, n_in, n_out, G, k):
    """Segments of a little more than a batch of 64 entries: their last batch holds a few quads, in streams of unequal length."""
    assert "walk_cells" in run_with_families(workloads.random_kan_layer(B + n_out, B, n_in, n_out, G, k, outside_frac=0.1))


@pytest.mark.parametrize("B,n_in,n_out,G,k", [(66000, 512, 259, 1000, 3), (66000, 1000, 130, 1000, 5)])
def test_quads_on_shared_partial_tables(B, n_in, n_out, G, k):
    """Tables whose nine partial slabs (half a gigabyte each) pass the budget, short enough for cell lists: the last chunk adds to
    what the first left in its slab, outputs two lanes share once.  Every run gives the same bits; an input's gradients depend on
    no other input, so three of them are compared with the oracle."""
    s = workloads.KanLayerSpec(n_in, n_out, G, k, -1.0, 1.0)
    gen = torch.Generator(device="cuda").manual_seed(B + n_in)
    rand = lambda std, *shape: torch.randn(shape, generator=gen, device="cuda") * std
    x = torch.rand((B, n_in), generator=gen, device="cuda") * 2.1 - 1.05
    coef, w_s, w_b, gy = rand(0.1, n_in, s.M, n_out), rand(1.0, n_in, n_out), rand(1.0, n_in, n_out), rand(B ** -0.5, B, n_out)
    seen = []
    hook = ctypes.CFUNCTYPE(None, ctypes.c_char_p, ctypes.c_void_p)(lambda family, stream: seen.append(family.decode()))
    none = ctypes.CFUNCTYPE(None, ctypes.c_char_p, ctypes.c_void_p)(lambda family, stream: None)
    binding.kan_set_launch_observer(hook, none)
    try:
        g = binding.kan_backward(s, x, coef, w_s, w_b, gy)
    finally:
        binding.kan_set_launch_observer(None, None)
    assert "walk_cells" in seen and seen.count("backward_walk") == 2       # eight or more chunks, then what is left
    again = binding.kan_backward(s, x, coef, w_s, w_b, gy)
    assert all(torch.equal(g[n], again[n]) for n in g)
    sel = [0, 7, n_in - 1]
    inv_h = oracle.inv_h_of(s.grid_lo, s.grid_hi, G)
    host = lambda t: np.ascontiguousarray(t.cpu().numpy())
    ref = oracle.kan_backward(host(x[:, sel]), host(coef[sel]), host(w_s[sel]), host(w_b[sel]), host(gy), G, k, s.grid_lo, inv_h)
    unit = 1.0 / float(inv_h)
    assert_close(g["gx"][:, sel].double() * unit, ref["gx"] * unit, GRAD_TOL, "gx")
    for n in ("gcoef", "gw_s", "gw_b"):
        assert_close(g[n][sel], ref[n], GRAD_TOL, n)


@pytest.mark.parametrize("B,n_in,n_out,G,k", [(9000, 9, 64, 100, 3), (3000, 33, 256, 40, 2), (5000, 9, 20, 64, 5), (2100, 33, 300, 30, 3)])
@pytest.mark.parametrize("lo,hi", [(0.5, 2.0), (-7.0, -3.0)])
def test_walk_over_padded_cells_of_a_grid_without_zero(B, n_in, n_out, G, k, lo, hi):
    """The pads between the cells are stored as x = 0, which lies outside these grids."""
    assert "walk_cells" in run_with_families(workloads.random_kan_layer(B + n_out, B, n_in, n_out, G, k, lo, hi, outside_frac=0.1))


MATRIX_SHAPES = [
    # sixteen positions an input, rows up to the last one; odd numbers of inputs, of outputs and of samples
    (12001, 37, 97, 10, 3), (12033, 64, 65, 13, 2), (12001, 40, 128, 14, 1),
    (12001, 33, 100, 15, 1), (12002, 39, 97, 20, 3),           # twenty-four: the first and the last row count
    (12001, 73, 127, 21, 3), (12031, 66, 130, 28, 3),          # thirty-two: the same
    (16001, 65, 256, 20, 3), (16001, 66, 255, 10, 3), (16001, 63, 193, 28, 2),      # sixty-four samples a workgroup
    (32700, 67, 300, 20, 3), (32641, 42, 512, 10, 3),          # a hundred and twenty-eight
    (12900, 139, 139, 29, 3), (5201, 231, 270, 38, 1), (5201, 232, 270, 38, 2), (12900, 137, 140, 44, 3),      # up to 47 rows
    (8096, 163, 230, 3, 4), (13457, 94, 136, 18, 5), (10900, 58, 123, 19, 5), (6801, 105, 161, 26, 5), (5200, 159, 446, 42, 5),      # windows of six
    (30001, 100, 417, 11, 4),
]


@pytest.mark.parametrize("B,n_in,n_out,G,k", MATRIX_SHAPES)
def test_matrix_forward(B, n_in, n_out, G, k):
    w = workloads.random_kan_layer(B + n_in, B, n_in, n_out, G, k, outside_frac=0.05)
    s, p = w.layers[0], w.params[0]
    x, coef, w_s, w_b = (dev(a) for a in (w.x, p["coef"], p["w_s"], p["w_b"]))
    y = []
    assert "forward_matrix" in families_of(lambda: y.append(binding.kan_forward(s, x, coef, w_s, w_b)))
    rows = np.r_[0:70, B // 2:B // 2 + 70, B - 200:B]
    ref = oracle.kan_forward(w.x[rows], p["coef"], p["w_s"], p["w_b"], G, k, s.grid_lo, oracle.inv_h_of(s.grid_lo, s.grid_hi, G))
    got = y[0].cpu().numpy()
    assert_close(y[0][torch.from_numpy(rows).cuda()], ref, 1e-5, "y")
    # in the 2-norm: up to 33 additions of partial sums and 3 products of leading parts an addition, each rounded to about half a
    # unit of 2^-24 of a sum that grows to the result: sqrt(4 * 33) / 2 * 0.6 units.  (One part of one factor lost: 4e-7 and more.)
    err = np.linalg.norm(got[rows] - ref) / np.linalg.norm(ref)
    assert err < 3.5 * 2.0 ** -24, err


@pytest.mark.parametrize("B,n_in,n_out,G,k", [(12001, 37, 97, 12, 3), (16001, 65, 256, 20, 3), (32700, 67, 300, 20, 3), (6801, 104, 161, 14, 5)])
def test_matrix_forward_keeps_infinities_apart(B, n_in, n_out, G, k):
    """Inputs and parameters that do not split into parts reach their own samples and outputs only."""
    w = workloads.random_kan_layer(B, B, n_in, n_out, G, k)
    s, p = w.layers[0], w.params[0]
    odd = [3, 64, 4100, B - 1]
    w.x[3, 2], w.x[64, 0], w.x[4100, n_in - 1], w.x[B - 1, 5] = np.inf, -np.inf, np.nan, 3e38
    p["coef"][7, G // 2, 5] = np.inf
    p["w_b"][9, n_out - 1] = np.nan
    p["coef"][n_in - 1, 3, 40] = 3e38
    x, coef, w_s, w_b = (dev(a) for a in (w.x, p["coef"], p["w_s"], p["w_b"]))
    y = []
    assert "forward_matrix" in families_of(lambda: y.append(binding.kan_forward(s, x, coef, w_s, w_b)))
    rows = np.r_[0:200, 4090:4110, B - 130:B]
    with np.errstate(all="ignore"):
        ref = oracle.kan_forward(w.x[rows], p["coef"], p["w_s"], p["w_b"], G, k, s.grid_lo, oracle.inv_h_of(s.grid_lo, s.grid_hi, G))
        got = y[0].cpu().numpy()[rows].astype(np.float64)
        ref = ref.astype(np.float32).astype(np.float64)         # past the range of a float: infinite
    assert np.isin(odd, rows).all() and not np.isfinite(ref[np.isin(rows, odd)]).all()
    assert np.array_equal(np.isnan(got), np.isnan(ref))
    big = ~np.isnan(ref) & ((np.abs(ref) > 1e30) | (np.abs(got) > 1e30))
    np.testing.assert_allclose(got[big], ref[big], rtol=1e-5)
    ok = ~np.isnan(ref) & ~big
    assert (np.abs(got[ok] - ref[ok]) <= 1e-5 * (1.0 + np.abs(ref[ok]))).all()
    assert ok.sum() > 0.8 * ok.size


def test_matrix_forward_workspace():
    """A workspace without room for the split table is refused, as before; the built-in scratch array takes the other kernel."""
    s = workloads.KanLayerSpec(560, 512, 20, 3, -1.0, 1.0)            # 27 MB folded, 69 with the split table
    B = 4096
    g = torch.Generator(device="cuda").manual_seed(3)
    x = torch.rand((B, s.n_in), generator=g, device="cuda") * 2 - 1
    coef, w_s, w_b = (torch.randn(d, generator=g, device="cuda") * 0.04 for d in ((s.n_in, s.M, s.n_out), (s.n_in, s.n_out), (s.n_in, s.n_out)))
    n = binding.kan_workspace_bytes(s, B, binding.PASS_FORWARD)
    with pytest.raises(binding.KanError):
        binding.kan_forward(s, x, coef, w_s, w_b, ws=torch.empty(n - 256, dtype=torch.uint8, device="cuda"))
    y = []
    assert "forward_matrix" in families_of(lambda: y.append(binding.kan_forward(s, x, coef, w_s, w_b)))
    z = torch.empty_like(y[0])
    assert n > binding.kan_static_scratch_bytes()
    assert "forward_matrix" not in families_of(lambda: binding.kan_forward_static(s, x, coef, w_s, w_b, z))
    assert ((z - y[0]).norm() / y[0].norm()).item() < 3e-6


@pytest.mark.parametrize("B,n_in,G,k,base", [
    (5001, 257, 30, 3, 1), (4099, 130, 12, 1, 1),              # a chunk's last list is short; a group of one and of two inputs
    (70000, 150, 1000, 3, 1),                                  # past what fits LDS: the other walk
    (33000, 40, 60, 3, 0), (70000, 33, 900, 2, 1),             # no base term; more cells than a wave has quads at a time
    (2048, 300, 1, 3, 1), (70000, 300, 5, 3, 1),               # one cell in the grid; cells that go on from wave to wave
])
def test_walk_of_one_output(B, n_in, G, k, base):
    w = workloads.random_kan_layer(B, B, n_in, 1, G, k, base_act=base, outside_frac=0.1)
    s, p = w.layers[0], w.params[0]
    _, g = run_layer_parity(w, gx_in_grid_units=G > 500)
    x, coef, w_s, w_b, gy = (dev(a) for a in (w.x, p["coef"], p["w_s"], p["w_b"], w.gy))
    again = binding.kan_backward(s, x, coef, w_s, w_b, gy)
    only = binding.kan_backward(s, x, coef, w_s, w_b, gy, want=("gcoef", "gw_s", "gw_b"))
    for n in ("gx", "gcoef", "gw_s", "gw_b"):
        assert torch.equal(g[n], again[n]), n
        assert n == "gx" or torch.equal(g[n], only[n]), n


def test_walk_of_one_output_keeps_infinities_apart():
    w = workloads.random_kan_layer(3, 9000, 64, 1, 40, 3)
    s, p = w.layers[0], w.params[0]
    w.gy[5, 0], w.gy[4000, 0] = np.inf, np.nan
    x, coef, w_s, w_b, gy = (dev(a) for a in (w.x, p["coef"], p["w_s"], p["w_b"], w.gy))
    g = binding.kan_backward(s, x, coef, w_s, w_b, gy)
    ref = oracle.kan_backward(w.x, p["coef"], p["w_s"], p["w_b"], w.gy, s.G, s.k, s.grid_lo, oracle.inv_h_of(s.grid_lo, s.grid_hi, s.G))
    for n in ("gx", "gcoef"):
        got, want = g[n].cpu().numpy(), ref[n]
        assert np.array_equal(np.isfinite(got), np.isfinite(want)), n
        ok = np.isfinite(want)
        assert ok.any() and not ok.all()
        assert (np.abs(got[ok] - want[ok]) <= GRAD_TOL * (1.0 + np.abs(want[ok]))).all(), n


@pytest.mark.parametrize("B,n_in,n_out,G,k,family", [
    (1280, 35, 1, 20, 3, "direct"), (1281, 35, 1, 20, 3, "narrow"), (513, 47, 1, 200, 2, "narrow"),     # one output, sixteen lanes a sample
    (131073, 33, 1, 20, 3, "narrow"), (9001, 31, 1, 20, 3, "narrow"),                                   # four
    (70001, 8, 16, 20, 3, "direct"), (70001, 33, 8, 20, 3, "direct"), (70001, 12, 8, 20, 3, "narrow"),  # wider
    (70001, 64, 5, 20, 3, "direct"), (70001, 63, 5, 20, 3, "narrow"), (70001, 33, 5, 256, 2, "direct"),
])
def test_narrow_lines(B, n_in, n_out, G, k, family):
    assert "forward_" + family in forward_with_families(workloads.random_kan_layer(n_in, B, n_in, n_out, G, k, outside_frac=0.02))
