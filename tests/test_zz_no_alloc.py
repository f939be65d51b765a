"""The allocation-free backward (dendsn_backward_noalloc, through the C ABI)
against the workspace backward (dendsn_backward) on the same inputs: every
output bit for bit, on two calls in a row, the second on a smaller layer (the
scratch array then still holds the first call's partials)."""

import numpy as np
import pytest

import paper_2412_06355_amd as dendsn
from tests.parity import announce, make_case, to_device

pytestmark = pytest.mark.gpu


def _cfg(**kw):
    base = dict(T=4, batch=2, C=256, S=1, B=4, beta=0.5, v_th=1.0, psi="mexhat", sg="sigmoid", sg_scale=4.0)
    base.update(kw)
    return dendsn.DendSNConfig(**base)


def _both(case, device):
    """Forward once, then the backward through both entry points."""
    import torch

    cfg = case.cfg
    d = to_device(case, device)
    spikes, _, ckpt = dendsn.forward(cfg, d["x"], d["alpha"], d["kappa"], d["xi"], d["zeta"], d["mask"],
                                     beta=d["beta"])
    ref = dendsn.backward(cfg, d["x"], d["alpha"], d["kappa"], d["xi"], d["zeta"], d["mask"], ckpt, d["gS"],
                          d["gV"], beta=d["beta"])
    out = {k: torch.full_like(v, float("nan")) for k, v in ref.items()}
    dendsn.dendsn_backward_noalloc(cfg, d["x"], d["alpha"], d["beta"], d["kappa"], d["xi"], d["zeta"], d["mask"],
                                   ckpt, d["gS"], d["gV"], out["grad_x"], out["grad_alpha"], out["grad_beta"],
                                   out["grad_kappa"], out["grad_xi"], out["grad_zeta"])
    torch.cuda.synchronize(device)
    return ref, out


def _bits(t):
    import torch

    return t.contiguous().view(torch.uint8)


def _assert_identical(ref, out):
    import torch

    for k in ref:
        assert torch.equal(_bits(ref[k]), _bits(out[k])), k


# a large layer first (12 MiB of partials: the gated fully connected shape),
# then smaller ones of other tilings
SEQUENCE = [
    ("fc-gated-large", dict(T=4, batch=64, C=8192, S=1, B=32), dict(mask_rho=0.5)),
    ("conv-small", dict(T=4, batch=2, C=16, S=1024, B=8), dict(random_affine=True)),
    ("long-ckpt-smaller", dict(T=24, batch=2, C=64, S=1, B=16, ckpt_every=8, beta=0.9),
     dict(x_mean=0.1, alpha=0.8, with_gv=True)),
]


def test_noalloc_backward_equals_workspace_backward(gpu_device):
    for name, ckw, mkw in SEQUENCE:
        cfg = _cfg(**ckw)
        assert dendsn.dendsn_bwd_workspace_bytes(cfg) <= dendsn.NOALLOC_SCRATCH_BYTES
        case = make_case(cfg, seed=3, name=f"noalloc/{name}", **mkw)
        announce(f"noalloc {name}: {cfg}")
        ref, out = _both(case, gpu_device)
        _assert_identical(ref, out)


@pytest.mark.parametrize("T,K", [(5, 0), (16, 8)])
def test_one_lane_where_two_would_outgrow_the_scratch(gpu_device, T, K):
    """Eight bf16 branches, more than four steps, so many tiles that two lanes a neuron
    would need more than the scratch array: the layer runs one lane a neuron, and the
    channels' gradients are those of a layer of few channels (two lanes)."""
    import torch

    few, reps = _cfg(T=T, batch=1, C=512, S=129, B=8, io="bf16", ckpt_every=K), 320
    many = few.with_(C=few.C * reps)
    case = make_case(few, seed=5, name=f"one lane T={T} K={K}", random_affine=True)
    announce(f"noalloc one lane: {many}")
    d = to_device(case, gpu_device)
    want, _ = _both(case, gpu_device)
    assert dendsn.dendsn_bwd_workspace_bytes(many) <= dendsn.NOALLOC_SCRATCH_BYTES
    x, gs = d["x"].repeat(1, reps, 1), d["gS"].repeat(1, reps)
    kappa, xi, zeta = (d[k].repeat(reps, 1) for k in ("kappa", "xi", "zeta"))
    _, _, ckpt = dendsn.forward(many, x, d["alpha"], kappa, xi, zeta, None)
    out = {k: torch.full_like(v.repeat(reps, 1) if v.dim() == 2 else v, float("nan"))
           for k, v in want.items() if k != "grad_x"}
    out["grad_x"] = torch.full_like(x, float("nan"))
    dendsn.dendsn_backward_noalloc(many, x, d["alpha"], None, kappa, xi, zeta, None, ckpt, gs, None, out["grad_x"],
                                   out["grad_alpha"], out["grad_beta"], out["grad_kappa"], out["grad_xi"],
                                   out["grad_zeta"])
    torch.cuda.synchronize(gpu_device)
    assert torch.equal(_bits(out["grad_x"]), _bits(want["grad_x"].repeat(1, reps, 1)))
    for k in ("grad_kappa", "grad_xi", "grad_zeta"):
        got = out[k].view(reps, few.C, -1)
        # a channel's T x 129 terms, in another order: a lane's T in a row and eight
        # levels of additions each way
        tol = 2 * (T + 8) * 2.0 ** -24 * (T * 129) ** 0.5 * want[k].abs().max()
        assert (got - want[k]).abs().max() <= tol, k
        assert torch.equal(got, got[:1].expand_as(got)), k


def test_noalloc_twice_on_a_shrinking_layer(gpu_device):
    """Two calls in a row, the second on a smaller layer of the same tiling."""
    for name, batch in (("first", 6), ("second-smaller", 2)):
        cfg = _cfg(T=8, batch=batch, C=96, S=300, B=8, ckpt_every=4)
        case = make_case(cfg, seed=9 + batch, x_std=1.2, alpha=0.6, mask_rho=0.6, name=f"noalloc/{name}")
        announce(f"noalloc {name}: {cfg}")
        ref, out = _both(case, gpu_device)
        _assert_identical(ref, out)
        assert np.isfinite(out["grad_x"].float().cpu().numpy()).all()


# A training step (forward, then the allocation-free backward) captured in a
# HIP graph through torch and replayed: every replay, with eager work and
# synchronisations between them, matches the eager step bit for bit.
def test_noalloc_step_under_graph_capture(gpu_device):
    import torch

    cfg = dendsn.DendSNConfig(T=8, batch=4, C=64, S=300, B=8, ckpt_every=4, beta=0.5, v_th=1.0, psi="mexhat",
                              sg="sigmoid", sg_scale=4.0)
    case = make_case(cfg, seed=21, mask_rho=0.6, with_gv=True, name="noalloc/graph")
    d = to_device(case, gpu_device)
    f32 = dict(dtype=torch.float32, device=gpu_device)
    spikes = torch.empty((cfg.T, cfg.N), **f32)
    ckpt = torch.empty((dendsn.dendsn_ckpt_bytes(cfg) // 4,), **f32)
    out = dict(grad_x=torch.empty_like(d["x"]), grad_alpha=torch.empty((1,), **f32),
               grad_beta=torch.empty((1,), **f32), grad_kappa=torch.empty((cfg.C, cfg.B), **f32),
               grad_xi=torch.empty((cfg.C, cfg.P), **f32), grad_zeta=torch.empty((cfg.C, cfg.B), **f32))

    def step():
        dendsn.dendsn_forward(cfg, d["x"], d["alpha"], d["beta"], d["kappa"], d["xi"], d["zeta"], d["mask"],
                              spikes, None, ckpt)
        dendsn.dendsn_backward_noalloc(cfg, d["x"], d["alpha"], d["beta"], d["kappa"], d["xi"], d["zeta"],
                                       d["mask"], ckpt, d["gS"], d["gV"], out["grad_x"], out["grad_alpha"],
                                       out["grad_beta"], out["grad_kappa"], out["grad_xi"], out["grad_zeta"])

    announce(f"graph capture of a noalloc step: {cfg}")
    step()  # eager (also looks up the scratch array's address before any capture)
    torch.cuda.synchronize(gpu_device)
    ref = {k: v.clone() for k, v in out.items()}
    ref["spikes"] = spikes.clone()

    side = torch.cuda.Stream(device=gpu_device)
    side.wait_stream(torch.cuda.current_stream(gpu_device))
    with torch.cuda.stream(side):
        step()
    torch.cuda.current_stream(gpu_device).wait_stream(side)
    torch.cuda.synchronize(gpu_device)

    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        step()
    torch.cuda.synchronize(gpu_device)

    bits = lambda t: t.contiguous().view(torch.uint8)
    for rep in range(3):
        for t in list(out.values()) + [spikes]:
            t.fill_(float("nan"))  # eager work between replays
        torch.cuda.synchronize(gpu_device)
        graph.replay()
        torch.cuda.synchronize(gpu_device)
        for k, v in out.items():
            assert torch.equal(bits(v), bits(ref[k])), (rep, k)
        assert torch.equal(bits(spikes), bits(ref["spikes"])), (rep, "spikes")
