"""Segmentation at the sizes where its kernels change over: position tiles of
the window sums, hidden sizes that end inside a column chunk, contexts hardly
longer than the window, the median in one workgroup and in passes, the warm-up
of the chunked recurrence.  Curvature against float64 (also where rows
alternate about a mean, which a quadratic form in the row differences gets
wrong by cancellation), scores against exact medians, slots against the serial
recurrence on the same scores."""
import pytest
import torch

from paper_2608_07001_amd import gracekv as gk

pytestmark = pytest.mark.gpu


def _hidden(T, Dh, n_seg, gen):
    topic = torch.randn(n_seg, T // 40 + 1, Dh, generator=gen, device="cuda").repeat_interleave(40, 1)[:, :T]
    return (topic + 1.5 * torch.randn(n_seg, T, Dh, generator=gen, device="cuda")).bfloat16()


def _run(T, Dh, n_seg, W=16, serial=False, seed=0, h=None):
    gen = torch.Generator(device="cuda").manual_seed(seed)
    cfg = gk.config_for(L=2, G=1, H=1, d=64, W=W, N_ctx=T - W, x=4.0 if T - W >= 64 else 1.5, dtype=gk.BF16, n_seg=n_seg, D_hidden=Dh,
                        flags=gk.FLAG_DP_SERIAL if serial else 0)
    buf = gk.allocate(cfg)
    buf.seg_ws.fill_(0xFF)                    # NaN wherever nothing was written
    if h is None:
        h = _hidden(T, Dh, n_seg, gen)
    s = torch.rand(T, generator=gen, device="cuda") * 8
    gk.segment(cfg, h, s, buf.kappa, buf.bscore, buf.slot_starts, buf.n_slots, buf.seg_ws)
    torch.cuda.synchronize()
    J = int(buf.n_slots.item())
    return cfg, h, s, buf.kappa[:T].double(), buf.bscore[:T].double(), buf.slot_starts[:J + 1].tolist(), buf.plan.N_c


def _kappa64(h):
    n_seg, T, _ = h.shape
    vals = []
    for x in h.double():
        x = x / x.norm(dim=-1, keepdim=True).clamp_min(1e-6)
        cs = torch.cat([torch.zeros_like(x[:1]), x.cumsum(0)])
        for w in (4, 8, 16):
            k = torch.zeros(T, dtype=torch.float64, device=x.device)
            i = torch.arange(w, max(T - w, w), device=x.device)
            a = x[i] - (cs[i + 1] - cs[i + 1 - w]) / w
            b = (cs[i + 1 + w] - cs[i + 1]) / w - x[i]
            k[i] = 1 - (a * b).sum(-1) / (a.norm(dim=-1).clamp_min(1e-6) * b.norm(dim=-1).clamp_min(1e-6))
            vals.append(k)
    vals = torch.stack(vals)
    return vals.mean(0) - 0.25 * vals.std(0, unbiased=False)


# kappa = 1 - cos: the dot product and the two norms each carry a few fp32 roundings of
# their value, about 5e-7 together for |cos| <= 1 (4e-7 seen); the line lies at four times
@pytest.mark.parametrize("T,Dh,n_seg,W", [(127, 40, 3, 16), (128, 32, 1, 16), (129, 264, 2, 1), (160, 8, 3, 8),
                                          (257, 72, 1, 37), (385, 4096, 1, 16), (500, 2048, 3, 16), (1031, 512, 3, 64),
                                          (70, 64, 8, 60), (90, 128, 3, 64), (33, 64, 1, 1), (4099, 1000, 2, 16)])
def test_curvature_tiles(T, Dh, n_seg, W):
    _, h, _, kappa, _, slots, N_c = _run(T, Dh, n_seg, W)
    err = float((kappa - _kappa64(h)).abs().max())
    print(f"T {T} Dh {Dh} n_seg {n_seg} N_c {N_c}: kappa off by {err:.2e}", flush=True)
    assert err < 2e-6
    assert slots[-1] == N_c


# 64 chunks of 512 ends, and 32768 values for the median
@pytest.mark.parametrize("T", [513 + 16, 32767, 32768, 32769, 32768 + 24, 32768 + 40, 33400])
def test_median_and_recurrence_changeover(T):
    _, _, s, kappa, b, slots, N_c = _run(T, 64, 1)
    z = 0.0
    for a, lam in ((kappa, 1.0), (s.double(), gk.default_config().lam_s)):
        med = a.sort().values[(T - 1) // 2]
        mad = (a.float() - med.float()).abs().sort().values[(T - 1) // 2].double()   # the fp32 deviations' own order
        z = z + lam * (a - med) / (1.4826 * mad + 1e-6)
    err = float((b - z).abs().max() / z.abs().max())
    print(f"T {T} N_c {N_c}: J {len(slots) - 1}, scores off by {err:.2e}", flush=True)
    assert err < 2e-6                         # a handful of fp32 roundings
    assert slots == _run(T, 64, 1, serial=True)[5]


# rows h_t = base + (-1)^t swing + noise: every window mean lies near the base, so
# kappa is well conditioned and window sums stay at a few fp32 roundings of it (1.1e-7
# rms), while sums over differences d_t = +-2 swing with weights up to the window
# cancel (1.1e-6 rms); the line lies at three times the former
@pytest.mark.parametrize("Dh", [512, 2048, 4096])
def test_curvature_of_alternating_rows(Dh):
    T = 1200
    gen = torch.Generator(device="cuda").manual_seed(Dh)
    sign = 1.0 - 2.0 * (torch.arange(T, device="cuda") % 2)
    base, swing = torch.randn(2, 3, 1, Dh, generator=gen, device="cuda")
    h = (base + 0.7 * sign[None, :, None] * swing + 0.2 * torch.randn(3, T, Dh, generator=gen, device="cuda")).bfloat16()
    err = (_run(T, Dh, 3, h=h)[3] - _kappa64(h)).pow(2).mean().sqrt()
    print(f"Dh {Dh}: kappa off by {float(err):.2e} (rms)", flush=True)
    assert err < 3e-7


# the tile of a position does not depend on the length of the context, nor do its sums
@pytest.mark.parametrize("T", [2000, 32640, 32768])
def test_curvature_independent_of_the_context_length(T):
    h = _hidden(33000, 1024, 3, torch.Generator(device="cuda").manual_seed(3))
    whole, part = _run(33000, 1024, 3, h=h)[3], _run(T, 1024, 3, h=h[:, :T].contiguous())[3]
    assert torch.equal(whole[:T - 16], part[:T - 16])


@pytest.mark.parametrize("N_c", [1, 2, 3, 15, 16, 17])
def test_contexts_of_a_few_tokens(N_c):
    # one slot takes them all below n_min + 1, and the terminal relaxation finds it
    gen = torch.Generator(device="cuda").manual_seed(N_c)
    cfg = gk.config_for(L=1, G=1, H=1, d=64, W=3, N_ctx=32 + N_c, x=1.0, dtype=gk.BF16, n_seg=2, D_hidden=64)
    buf = gk.allocate(cfg)
    assert buf.plan.N_c == N_c
    buf.seg_ws.fill_(0xFF)
    T = buf.plan.T
    h, s = _hidden(T, 64, 2, gen), torch.rand(T, generator=gen, device="cuda") * 8
    gk.segment(cfg, h, s, buf.kappa, buf.bscore, buf.slot_starts, buf.n_slots, buf.seg_ws)
    J = int(buf.n_slots.item())
    assert buf.slot_starts[:J + 1].tolist() == [0, N_c]
