"""Edge sizes of the kernels' tiles, remainders and dispatch lines, against the CPU oracle (bars as in test_gpu_kan)."""
import pytest
import torch

from paper_2408_11200_amd import binding, workloads
from test_gpu_kan import dev, run_layer_parity

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B,n_in,n_out,G,k", [
    (1, 1, 1, 1, 1),                   # one pair
    (5, 31, 16, 3, 3),                 # four waves, exactly one 16-lane tile
    (3, 33, 17, 10, 2),                # sixteen waves, ragged 32-lane tile
    (2, 1100, 33, 4, 3),               # more inputs than one round of pair evaluations, ragged 64-lane tile
    (2049, 40, 65, 6, 3),              # four samples per workgroup, ragged batch, two tiles of one output per lane
    (2050, 35, 126, 6, 3),             # two outputs per lane
    (9, 70, 130, 12, 5), (2047, 20, 64, 5, 4),      # window of six rows
    (4096, 10, 64, 8, 3), (4097, 10, 64, 8, 3),     # the last batch of the direct kernel and the first past it
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
