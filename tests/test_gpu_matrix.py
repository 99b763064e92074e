"""The matrix-core forward kernel and the kernels beside it at the ends of the float range, and their sums' accuracy."""
import numpy as np
import pytest
import torch

import oracle
from paper_2408_11200_amd import binding, workloads
from test_gpu_edges import families_of
from test_gpu_kan import dev

pytestmark = pytest.mark.gpu


def run_rows(w, rows, family):
    """The layer's outputs at some rows and the oracle's, on the kernel family that is meant."""
    s, p = w.layers[0], w.params[0]
    x, coef, w_s, w_b = (dev(a) for a in (w.x, p["coef"], p["w_s"], p["w_b"]))
    y = []
    assert "forward_" + family in families_of(lambda: y.append(binding.kan_forward(s, x, coef, w_s, w_b)))
    with np.errstate(all="ignore"):
        ref = oracle.kan_forward(w.x[rows], p["coef"], p["w_s"], p["w_b"], s.G, s.k, s.grid_lo, oracle.inv_h_of(s.grid_lo, s.grid_hi, s.G))
    return y[0].cpu().numpy()[rows].astype(np.float64), ref


def rel(got, ref):
    return np.linalg.norm(got - ref) / np.linalg.norm(ref)


def chain_bound(chain, parts):
    """2-norm error of a sum of `parts` partial sums of `chain` terms each, all one behind another, in the mean: an addition rounds to
    0.42 * 2^-24 of its sum and the sums grow like the root of their terms, which makes 0.42 * sqrt((chain + parts) / 2); the
    weights and base values come with 0.7.  A sixth is left for what the terms of a layer differ."""
    return 1.16 * np.hypot(0.42 * np.sqrt((chain + parts) / 2), 0.7) * 2.0 ** -24


# one form each: 64 samples a workgroup with four and eight tiles, 128; windows of six
MATRIX_FORMS = [(12001, 37, 97, 12, 3), (16001, 65, 256, 20, 3), (32700, 67, 300, 20, 3), (6801, 104, 161, 14, 5)]


@pytest.mark.parametrize("B,n_in,n_out,G,k", MATRIX_FORMS)
def test_matrix_forward_overflows_to_infinity(B, n_in, n_out, G, k):
    """Factors that split and a product that is past the range of a float, or up to its last percent: as in plain fp32."""
    w = workloads.random_kan_layer(B + 1, B, n_in, n_out, G, k)
    p = w.params[0]
    g = np.random.default_rng(3)
    rows = np.r_[0:160, B - 70:B]
    for n, b in enumerate(rows[::3]):
        w.x[b, n % 7] = 10.0 ** g.uniform(24, 34)               # an input of each of these samples, on large weights of either sign
    p["w_b"][:7] = 10.0 ** g.uniform(12, 16, (7, n_out)) * g.choice([-1.0, 1.0], (7, n_out))
    w.x[rows[1]] = 0.0
    w.x[rows[1], 0], p["w_b"][0, 3] = 1e20, 3.38e18             # 0.993 of the largest float
    got, ref = run_rows(w, rows, "matrix")
    with np.errstate(all="ignore"):
        ref = ref.astype(np.float32).astype(np.float64)
    assert not np.isnan(ref).any() and np.isinf(ref).sum() > 1000 and np.isfinite(ref[1, 3])
    assert np.array_equal(np.isinf(got), np.isinf(ref)) and np.array_equal(got[np.isinf(ref)], ref[np.isinf(ref)])
    ok = np.isfinite(ref)
    np.testing.assert_allclose(got[ok], ref[ok], rtol=1e-5, atol=1e-5 * np.abs(p["w_b"][:7]).max())


@pytest.mark.parametrize("B,n_in,n_out,G,k", MATRIX_FORMS)
def test_matrix_forward_of_small_values(B, n_in, n_out, G, k):
    """Parameters whose lower parts are below the smallest bf16 number keep their 24 bits."""
    w = workloads.random_kan_layer(B + 2, B, n_in, n_out, G, k)
    p = w.params[0]
    p["coef"] = (p["coef"] * 2.0 ** -112).astype(np.float32)
    p["w_b"] = (p["w_b"] * 2.0 ** -112).astype(np.float32)
    rows = np.r_[0:70, B - 70:B]
    got, ref = run_rows(w, rows, "matrix")
    assert rel(got, ref) < 3.5 * 2.0 ** -24


def test_matrix_forward_beside_values_that_do_not_split():
    """The other outputs of a tile with an infinite parameter are summed as accurately as ever."""
    B, n_in, n_out, G, k = 9001, 400, 100, 12, 3
    w = workloads.random_kan_layer(5, B, n_in, n_out, G, k)
    w.params[0]["w_b"][7, 33] = np.inf
    rows = np.r_[0:70, B - 70:B]
    got, ref = run_rows(w, rows, "matrix")
    cols = np.r_[32:33, 34:64]
    assert rel(got[:, cols], ref[:, cols]) < chain_bound(5 * 32, 13)


@pytest.mark.parametrize("B,n_in,n_out,G,k,family,chain,parts", [
    (16510, 403, 164, 19, 1, "matrix", 75, 16), (18893, 169, 141, 8, 2, "matrix", 42, 16), (18327, 243, 158, 16, 3, "matrix", 76, 16),
    (5074, 23, 332, 36, 5, "matrix", 10, 16), (8161, 16, 256, 9, 5, "matrix", 7, 16), (8245, 32, 128, 8, 5, "matrix", 14, 16),
    (19696, 25, 83, 5, 3, "lds_rows", 8, 16), (30106, 43, 93, 32, 3, "lds_rows", 14, 16), (26437, 74, 85, 80, 3, "lds_rows", 24, 16),
    (22677, 64, 128, 134, 5, "lds_rows", 28, 16), (21483, 238, 105, 62, 1, "lds_rows", 45, 16),
    (2422, 700, 1, 20, 3, "narrow", 55, 64),
    (60000, 64, 16, 20, 3, "direct", 5, 15),            # 64 groups, eight in pairs and the eights in a row: three levels and 8 / 2 of them
])
def test_forward_sums(B, n_in, n_out, G, k, family, chain, parts):
    """No longer sums than those of the direct kernel, whose groups of lanes, sixteen or 64, share the inputs."""
    rows = np.r_[0:100, B - 100:B]
    got, ref = run_rows(workloads.random_kan_layer(B, B, n_in, n_out, G, k), rows, family)
    err = rel(got, ref)
    assert err < chain_bound(chain, parts), err * 2 ** 24


@pytest.mark.parametrize("B,n_in,n_out,G,k,family", [
    (2182, 512, 256, 16, 3, "direct"),                          # its table past L2: 198 us, on the matrix cores 228
    (33091, 96, 44, 179, 1, "direct"), (38374, 96, 40, 243, 5, "direct"),       # tiles of 32 on eight waves: 145 / 158, 222 / 266
    (40000, 98, 38, 202, 3, "lds_rows"), (51421, 98, 38, 202, 4, "lds_rows"),   # them: direct 168 / 156, 309 / 269
])
def test_layers_left_to_the_other_kernels(B, n_in, n_out, G, k, family):
    got, ref = run_rows(workloads.random_kan_layer(B, B, n_in, n_out, G, k), np.r_[0:50, B - 50:B], family)
    assert rel(got, ref) < 1e-6


def layer_tensors(B, s):
    g = torch.Generator(device="cuda").manual_seed(3)
    x = torch.rand((B, s.n_in), generator=g, device="cuda") * 2 - 1
    return [x] + [torch.randn(d, generator=g, device="cuda") * 0.04 for d in ((s.n_in, s.M, s.n_out), (s.n_in, s.n_out), (s.n_in, s.n_out))]


def test_matrix_forward_in_a_workspace_of_the_folded_table():
    """The split table is counted only for the batches that the kernel takes, and a workspace without it serves them on another kernel."""
    s = workloads.KanLayerSpec(512, 512, 20, 3, -1.0, 1.0)
    folded = s.n_in * (s.M + 1) * s.n_out * 4
    assert binding.kan_workspace_bytes(s, 64, binding.PASS_FORWARD) == folded
    assert binding.kan_workspace_bytes(s, 4096, binding.PASS_FORWARD) > 2 * folded
    x, coef, w_s, w_b = layer_tensors(4096, s)
    y, ws = [], torch.empty(folded, dtype=torch.uint8, device="cuda")
    assert "forward_matrix" in families_of(lambda: y.append(binding.kan_forward(s, x, coef, w_s, w_b)))
    assert "forward_matrix" not in families_of(lambda: y.append(binding.kan_forward(s, x, coef, w_s, w_b, ws=ws)))
    assert ((y[1] - y[0]).norm() / y[0].norm()).item() < 3e-6
    assert torch.equal(ws.view(torch.float32), torch.cat([coef * w_s[:, None, :], w_b[:, None, :]], dim=1).flatten())
    with pytest.raises(binding.KanError):
        binding.kan_forward(s, x, coef, w_s, w_b, ws=ws[:folded - 256])


@pytest.mark.parametrize("B,n_in,n_out,G,k,family", [
    (4096, 560, 512, 20, 3, "forward_matrix_range"),        # a split table of 42 MB: rounds of eight tiles
    (4099, 1100, 225, 20, 3, "forward_matrix_range"),       # of five and three
    (5003, 2700, 97, 8, 5, "forward_matrix_range"),         # of two, windows of six
    (12001, 37, 97, 12, 3, "forward_matrix"),               # whole
])
def test_matrix_forward_in_the_static_array(B, n_in, n_out, G, k, family):
    """The same bits as kan_forward, also where the split table does not fit the array, and of values that do not split."""
    s = workloads.KanLayerSpec(n_in, n_out, G, k, -1.0, 1.0)
    x, coef, w_s, w_b = layer_tensors(B, s)
    y, z = torch.empty((B, n_out), device="cuda"), torch.empty((B, n_out), device="cuda")
    for special in (False, True):
        if special:
            x[5, 3], x[B - 1, 2], coef[7, 2, n_out - 1], w_b[4, 40] = float("inf"), 1e30, float("inf"), 1e12
        z.zero_()
        assert "forward_matrix" in families_of(lambda: binding.kan_forward(s, x, coef, w_s, w_b, y=y))
        assert family in families_of(lambda: binding.kan_forward_static(s, x, coef, w_s, w_b, z))
        assert torch.equal(y.view(torch.int32), z.view(torch.int32))


@pytest.mark.parametrize("B,n_in,G,k", [(3000, 64, 5, 1), (2011, 33, 9, 2), (4001, 50, 3, 3), (5000, 20, 3, 1), (140000, 36, 1, 3), (2300, 48, 1, 2)])
def test_one_output_windows_over_the_ends(B, n_in, G, k):
    """Windows that hang over an end of the table, samples off the grid, and infinite parameters that only the samples of
    their windows meet."""
    w = workloads.random_kan_layer(B + n_in, B, n_in, 1, G, k, outside_frac=0.3)
    s, p = w.layers[0], w.params[0]
    rows = np.r_[0:400, B - 400:B]
    got, ref = run_rows(w, rows, "narrow")
    assert rel(got, ref) < 4 * 2.0 ** -24
    p["coef"][3, 0, 0], p["coef"][5, s.M - 1, 0] = np.inf, -np.inf
    got, ref = run_rows(w, rows, "narrow")
    near, touched = np.zeros(len(rows), bool), np.zeros(len(rows), bool)        # in the four rows of a window, in its k + 1
    for i, row in ((3, 0), (5, s.M - 1)):
        cell = np.floor((w.x[rows, i].astype(np.float64) + 1) * G / 2)
        near |= (cell <= row) & (row <= cell + 3)
        touched |= (cell <= row) & (row <= cell + k)
    assert touched.any() and not np.isfinite(got[touched]).any()
    assert np.isfinite(got[~near]).all()
    assert near.all() or rel(got[~near], ref[~near]) < 4 * 2.0 ** -24
