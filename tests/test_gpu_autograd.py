"""The autograd glue hands autograd exactly what the C-ABI calls return, and a small stack trains."""
import numpy as np
import pytest
import torch

import oracle
from paper_2408_11200_amd import autograd, binding, workloads

pytestmark = pytest.mark.gpu


def dev(a, grad=False):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda().requires_grad_(grad)


def test_kan_stack_gradients_through_autograd_match_oracle():
    """[2,5,1] with the MSE loss: torch chains the two layers, the oracle chains them in fp64."""
    w = workloads.config1()
    S, P = w.layers, w.params
    T = [{n: dev(a, True) for n, a in p.items()} for p in P]
    x = dev(w.x)
    h = autograd.kan_layer(S[0], x, T[0]["coef"], T[0]["w_s"], T[0]["w_b"])
    y = autograd.kan_layer(S[1], h, T[1]["coef"], T[1]["w_s"], T[1]["w_b"])
    loss = ((y - dev(w.target)) ** 2).mean()
    loss.backward()
    ih = [oracle.inv_h_of(s.grid_lo, s.grid_hi, s.G) for s in S]
    hn, yn = h.detach().cpu().numpy(), y.detach().cpu().numpy()
    gy = (2.0 / yn.size) * (yn.astype(np.float64) - w.target)
    r2 = oracle.kan_backward(hn, P[1]["coef"], P[1]["w_s"], P[1]["w_b"], np.float32(gy), 5, 3, -1.0, ih[1])
    r1 = oracle.kan_backward(w.x, P[0]["coef"], P[0]["w_s"], P[0]["w_b"], np.float32(r2["gx"]), 5, 3, -1.0, ih[0])
    for l, r in ((0, r1), (1, r2)):
        for name, key in (("coef", "gcoef"), ("w_s", "gw_s"), ("w_b", "gw_b")):
            got = T[l][name].grad.cpu().numpy().astype(np.float64)
            err = np.abs(got - r[key]) / (1.0 + np.abs(r[key]))
            assert err.max() <= 1e-4, (l, name, err.max())


def test_adam_reduces_the_regression_loss():
    """A few hundred Adam steps on y = sin(pi x0) + x1^2 with the [2,5,1] network."""
    w = workloads.config1()
    S = w.layers
    T = [{n: dev(a, True) for n, a in p.items()} for p in w.params]
    x, target = dev(w.x), dev(w.target)
    opt = torch.optim.Adam([t for layer in T for t in layer.values()], lr=2e-2)
    losses = []
    for _ in range(300):
        opt.zero_grad()
        h = autograd.kan_layer(S[0], x, T[0]["coef"], T[0]["w_s"], T[0]["w_b"])
        y = autograd.kan_layer(S[1], h, T[1]["coef"], T[1]["w_s"], T[1]["w_b"])
        loss = ((y - target) ** 2).mean()
        loss.backward()
        opt.step()
        losses.append(float(loss.detach()))
    assert losses[-1] < 0.05 * losses[0], (losses[0], losses[-1])


def test_ukan_layer_gradients_through_autograd():
    rng = np.random.default_rng(4)
    spec = workloads.UkanLayerSpec(6, 32, 3, 0.25, 8, 8, 16)
    p = workloads.ukan_params(rng, spec)
    x = np.float32(rng.standard_normal((500, 6)) * 2.0)
    gy = np.float32(rng.standard_normal((500, 32)) / np.sqrt(500))
    T = {n: dev(a, True) for n, a in p.items() if n != "w_b"}
    xt = dev(x, True)
    y = autograd.ukan_layer(spec, xt, T, 64)
    y.backward(dev(gy))
    ref = oracle.ukan_backward(x, p, gy, 3, oracle.inv_h_of_spacing(spec.h))
    pairs = [("gx", xt)] + [("g" + n, T[n]) for n in ("E", "W1", "b1", "W2", "b2", "scale")]
    for key, t in pairs:
        got = t.grad.cpu().numpy().astype(np.float64)
        err = np.abs(got - ref[key]) / (1.0 + np.abs(ref[key]))
        assert err.max() <= 1e-4, (key, err.max())


def kan_tensors(B=300, n_in=5, n_out=7):
    w = workloads.random_kan_layer(11, B, n_in, n_out, 9, 3)
    return w.layers[0], dev(w.x, True), {n: dev(a, True) for n, a in w.params[0].items()}, dev(w.gy)


def test_nodes_keep_autograd_contracts():
    """What a program may do around a node: hooks on its saved tensors, inputs that need no gradient, views, changes in place
    between the passes, a second derivative, wrong tensors."""
    s, x, p, gy = kan_tensors()
    layer = lambda x, p: autograd.kan_layer(s, x, p["coef"], p["w_s"], p["w_b"])
    names = ("coef", "w_s", "w_b")
    want = binding.kan_backward(s, x.detach(), *(p[n].detach() for n in names), gy)
    seen = []
    with torch.autograd.graph.saved_tensors_hooks(lambda t: seen.append(t.shape) or t.cpu(), lambda t: t.cuda()):
        y = layer(x, p)
    assert len(seen) == 5                                               # x, the parameters and the folded table
    g = torch.autograd.grad(y, [x] + [p[n] for n in names], gy)
    assert all(torch.equal(a, want[n]) for a, n in zip(g, ("gx", "gcoef", "gw_s", "gw_b")))
    only = torch.autograd.grad(layer(x.detach(), {n: p[n] if n == "w_s" else p[n].detach() for n in names}), p["w_s"], gy)[0]
    assert torch.equal(only, want["gw_s"])
    xt = x.detach().t().contiguous().t().requires_grad_(True)           # another order of strides
    assert torch.equal(torch.autograd.grad(layer(xt, p), xt, gy)[0], want["gx"])
    assert not layer(x.detach(), {n: t.detach() for n, t in p.items()}).requires_grad
    with torch.no_grad():
        assert layer(x, p).grad_fn is None
    y = layer(x, p)
    with torch.no_grad():
        p["w_s"].mul_(2.0)
    with pytest.raises(RuntimeError, match="modified by an inplace operation"):
        y.backward(gy)
    first = torch.autograd.grad(layer(x, p), x, gy, create_graph=True)[0]
    assert not first.requires_grad                                      # no second derivative is claimed
    with pytest.raises(AssertionError):
        layer(x.double(), p)
    with pytest.raises(AssertionError):
        layer(x.detach().cpu(), {n: t.detach().cpu() for n, t in p.items()})
    with pytest.raises(RuntimeError):
        torch.func.vmap(lambda a: layer(a, p))(x.detach().reshape(3, 100, 5))
    bad = workloads.KanLayerSpec(s.n_in, s.n_out, s.G, 6, -1.0, 1.0)
    with pytest.raises(binding.KanError) as e:
        autograd.kan_layer(bad, x, p["coef"], p["w_s"], p["w_b"])
    assert e.value.status == binding.KAN_ERR_UNSUPPORTED


@pytest.mark.parametrize("unpack", [lambda t: t.cpu(), lambda t: torch.stack((t, t), 1)[:, 0]])
def test_what_a_forward_pass_left_is_checked_again(unpack):
    """The folded table and the UKAN intermediates go through the hooks on saved tensors: one that comes back on the host or
    with gaps is refused, as binding.py refuses it."""
    s, x, p, gy = kan_tensors()
    rng = np.random.default_rng(4)
    spec = workloads.UkanLayerSpec(3, 4, 3, 0.25, 8, 8, 16)
    T = {n: dev(a, True) for n, a in workloads.ukan_params(rng, spec).items() if n != "w_b"}
    xu = dev(np.float32(rng.uniform(-1, 1, (100, 3))), True)
    with torch.autograd.graph.saved_tensors_hooks(lambda t: t, lambda t: unpack(t) if t.dtype == torch.uint8 else t):
        outs = [autograd.kan_layer(s, x, p["coef"], p["w_s"], p["w_b"]), autograd.ukan_layer(spec, xu, T, 64)]
    for y in outs:
        with pytest.raises(AssertionError):
            y.sum().backward()


def test_nodes_run_on_the_stream_of_their_forward_pass():
    s, x, p, gy = kan_tensors(B=2000, n_in=16, n_out=20)
    names = ("coef", "w_s", "w_b")
    want = binding.kan_backward(s, x.detach(), *(p[n].detach() for n in names), gy)
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        y = autograd.kan_layer(s, x, p["coef"], p["w_s"], p["w_b"])
    g = torch.autograd.grad(y, [x] + [p[n] for n in names], gy)
    torch.cuda.synchronize()
    assert all(torch.equal(a, want[n]) for a, n in zip(g, ("gx", "gcoef", "gw_s", "gw_b")))


def test_ukan_node_reports_a_span_past_the_bound():
    rng = np.random.default_rng(4)
    spec = workloads.UkanLayerSpec(3, 4, 3, 0.25, 8, 8, 16)
    T = {n: dev(a) for n, a in workloads.ukan_params(rng, spec).items() if n != "w_b"}
    x = dev(np.float32(rng.uniform(-50, 50, (100, 3))))
    with pytest.raises(binding.KanError) as e:
        autograd.ukan_layer(spec, x, T, 8)
    assert e.value.status == binding.KAN_ERR_RANGE


class Layers(torch.nn.Module):
    """A UKAN layer on top of a KAN layer, its parameters the module's own."""

    def __init__(self, kan, p, ukan, q):
        super().__init__()
        self.specs = (kan, ukan)
        own = lambda p: torch.nn.ParameterDict({n: torch.nn.Parameter(t.detach().clone()) for n, t in p.items()})
        self.p, self.q = own(p), own(q)

    def forward(self, x):
        h = autograd.kan_layer(self.specs[0], x, self.p["coef"], self.p["w_s"], self.p["w_b"])
        return autograd.ukan_layer(self.specs[1], h, dict(self.q.items()), 256)


def test_traced_module_runs_the_layers(tmp_path):
    """torch.jit.trace records the layers: the traced module gives the module's own bits on inputs that the trace has not seen,
    trains, and can be saved; parameters that are no part of the module are refused as for any operator."""
    s, x, p, _ = kan_tensors()
    spec = workloads.UkanLayerSpec(s.n_out, 4, 3, 0.5, 8, 8, 16)
    q = {n: dev(a) for n, a in workloads.ukan_params(np.random.default_rng(4), spec).items() if n != "w_b"}
    m = Layers(s, p, spec, q)
    traced = torch.jit.trace(m, (x.detach(),))
    traced.save(str(tmp_path / "layers.pt"))
    loaded = torch.jit.load(str(tmp_path / "layers.pt"))
    for scale in (0.5, 0.25, 1.0):
        xs = (x.detach() * scale).requires_grad_(True)
        want = m(xs)
        assert torch.equal(traced(xs), want) and torch.equal(loaded(xs), want)
        leaves = [xs] + list(m.parameters())
        for a, b in zip(torch.autograd.grad(traced(xs).sum(), leaves), torch.autograd.grad(want.sum(), leaves)):
            assert torch.equal(a, b)
    with pytest.raises(RuntimeError, match="requires grad"):
        torch.jit.trace(lambda a: autograd.kan_layer(s, a, p["coef"], p["w_s"], p["w_b"]), (x.detach(),))


def test_kan_node_keeps_the_folded_table_only():
    """What the forward pass needs besides is given back when it ends: 128 -> 96 on the matrix-core kernel, whose split table is the larger."""
    s, x, p, gy = kan_tensors(12001, 128, 96)
    folded = binding.kan_workspace_bytes(s, 0, binding.PASS_FORWARD)
    assert binding.kan_workspace_bytes(s, 12001, binding.PASS_FORWARD) > 2 * folded
    held = []
    with torch.autograd.graph.saved_tensors_hooks(lambda t: held.append((t.dtype, t.untyped_storage().nbytes())) or t, lambda t: t):
        y = autograd.kan_layer(s, x, p["coef"], p["w_s"], p["w_b"])
    assert [n for dtype, n in held if dtype == torch.uint8] == [folded]
    assert torch.equal(y, binding.kan_forward(s, x.detach(), *(p[n].detach() for n in ("coef", "w_s", "w_b"))))
    g = torch.autograd.grad(y, [x, p["coef"]], gy)
    want = binding.kan_backward(s, x.detach(), *(p[n].detach() for n in ("coef", "w_s", "w_b")), gy)
    assert torch.equal(g[0], want["gx"]) and torch.equal(g[1], want["gcoef"])
