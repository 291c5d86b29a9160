"""Gates whose summed grid is not expanded (a NaN or infinite sample, powers
beyond the FP32 range): redone by direct transforms or matrix products, split over
the chip, beside gates that are not affected."""

import numpy as np
import pytest

torch = pytest.importorskip("torch")

from oracle import integrate_spectra as oracle_spectra  # noqa: E402
from synth import random_inputs  # noqa: E402
from tests.conftest import ensure_library  # noqa: E402
from tests.parity_util import assert_spectra_match  # noqa: E402

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.fixture(scope="module")
def ispl():
    ensure_library()
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a GPU")
    import paper_2311_18737_amd as pkg

    return pkg


def best_us(call, reps=6):
    call()
    torch.cuda.synchronize()
    best = float("inf")
    for _ in range(reps):
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        a.record()
        call()
        b.record()
        torch.cuda.synchronize()
        best = min(best, a.elapsed_time(b) * 1e3)
    return best


CASES = [
    # N,     L,    G,   P,   code kind, zoom
    (16384, 1000, 300, 400, "bpsk", False),
    (8192, 300, 400, 400, "phase", False),
    (32768, 2000, 150, 200, "phase", False),
    (16384, 3000, 150, 200, "bpsk", False),  # sign bits, LDS copies
    (16384, 256, 300, 400, "bpsk", True),
    (16384, 700, 200, 300, "phase", True),
]


@pytest.mark.parametrize("case", CASES, ids=lambda c: "N{}_L{}_G{}_P{}_{}_zoom{}".format(*c))
@pytest.mark.parametrize("value", [np.nan, np.inf])
def test_one_bad_sample(ispl, case, value):
    """The gates that read the sample are not finite in any bin, the others exactly as without it,
    and the call takes no more than a few times as long as a clean one (the bad gates' direct
    transforms, a launch or two each, at any pulse count)."""
    N, L, G, P, kind, zoomed = case
    print(f"case {case} {value}", flush=True)
    step = L // 2
    stride = (G - 1) * step + L
    samples, tx = random_inputs(P, stride, L, code_kind=kind, seed=N + L)
    bad = samples.copy()
    bad[P // 3, 10 * step + 1] = value  # read by gates 9 and 10
    ctx = ispl.Context(code_len=L, fft_len=N, n_gates=G, gate_step=step, pulse_stride=stride,
                       max_pulses=P)
    xt = torch.from_numpy(tx).to(DEV)
    clean, broken = (torch.from_numpy(s).to(DEV) for s in (samples, bad))
    if zoomed:
        zoom = ispl.Zoom(ctx, 256, "fp16x3")
        start = torch.arange(G, dtype=torch.int32, device=DEV) * 97
        call = lambda x, out: zoom.spectra(x, xt, start, out=out)  # noqa: E731
    else:
        call = lambda x, out: ctx.integrate_spectra(x, xt, out=out)  # noqa: E731
    width = 256 if zoomed else N
    want, got = (torch.empty((G, width), device=DEV) for _ in range(2))
    t_clean = best_us(lambda: call(clean, want))
    t_bad = best_us(lambda: call(broken, got))
    hit = torch.zeros(G, dtype=torch.bool, device=DEV)
    hit[9:11] = True
    assert not torch.isfinite(got[hit]).any()
    assert torch.equal(got[~hit], want[~hit]) and torch.isfinite(want).all()
    print(f"clean {t_clean:.0f} us, with a bad sample {t_bad:.0f} us", flush=True)
    assert t_bad <= 3.0 * t_clean + 100.0
    if zoomed:
        zoom.close()
    ctx.close()


@pytest.mark.parametrize("case", [
    # N,     L,   G,  P,  type, code per pulse, kind
    (16384, 600, 96, 200, "c64", True, "bpsk"),
    (4096, 100, 300, 50, "c64", False, "phase"),
    (65536, 500, 8, 60, "c64", True, "bpsk"),
    (32768, 3000, 24, 40, "c64", True, "bpsk"),
    (16384, 1500, 60, 30, "c64", False, "phase"),
], ids=lambda c: "N{}_L{}_G{}_P{}_{}_{}_{}".format(*c))
def test_redone_gates_match_oracle(ispl, case):
    """Gates that overflow in one pulse's line (redone in FP32), among others, with and without a
    gate list and accumulation."""
    N, L, G, P, st, per, kind = case
    step = L
    stride = G * step
    samples, tx = random_inputs(P, stride, L, sample_type=st, code_kind=kind,
                                tx_rows=None if per else 1, seed=N + L)
    hot = [0, 3, G // 2, G - 1]
    n = np.arange(L)
    for g in hot:  # one point of the line's grid beyond FP32, the bins below it finite
        code = tx[1] if per else tx[0]
        samples[1, g * step:(g + 1) * step] += (2.5e19 / L * np.exp(2j * np.pi * 0.125 * n) * code
                                                ).astype(np.complex64)
    with np.errstate(all="ignore"):
        ref = oracle_spectra(samples, tx, n_gates=G, gate_step=step, first_gate=0, fft_len=N,
                             tx_per_pulse=per)
    ctx = ispl.Context(code_len=L, fft_len=N, n_gates=G, gate_step=step, pulse_stride=stride,
                       sample_type=st, max_pulses=P)
    xs, xt = torch.from_numpy(samples).to(DEV), torch.from_numpy(tx).to(DEV)
    out = ctx.integrate_spectra(xs, xt)
    got = out.cpu().numpy().astype(np.float64)
    others = [g for g in range(G) if g not in hot]
    assert_spectra_match(got[others], ref[others], what="gates beside")
    big = float(np.finfo(np.float32).max)
    for g in hot:
        over, under = ref[g] > 1.0001 * big, ref[g] < 0.9999 * big
        assert over.any() and np.isinf(got[g][over]).all() and np.isfinite(got[g][under]).all()
    cool = torch.ones(G, dtype=torch.bool, device=DEV)
    cool[hot] = False
    twice = ctx.integrate_spectra(xs, xt, out=out.clone(), accumulate=True)
    assert torch.equal(twice, out + out)
    lst = torch.arange(G - 1, -1, -1, dtype=torch.int32, device=DEV)
    part = torch.full((G, N), -1.0, device=DEV)
    keep = G - 2  # leaves out gates 0 and 1
    ctx.integrate_spectra(xs, xt, out=part,
                          gates=(lst, torch.tensor([keep], dtype=torch.int32, device=DEV)))
    assert bool((part[:2] == -1.0).all())
    sel = cool.clone()
    sel[:2] = False
    assert torch.equal(part[sel], out[sel])
    np.testing.assert_allclose(part[hot[1:]].cpu().numpy(), out[hot[1:]].cpu().numpy(), rtol=1e-5)
    ctx.close()
