"""Accuracy of spectra with one narrow line per tested gate, where a summed grid
is expanded: rounding at a line's grid points is spread over the gate's bins, in
proportion to the line's height over the mean.

Every error is relative to max(S, mean S) of the FP64 oracle's spectrum."""

import numpy as np
import pytest

torch = pytest.importorskip("torch")

from oracle import integrate_spectra as oracle_spectra  # noqa: E402
from tests.conftest import ensure_library  # noqa: E402

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.fixture(scope="module")
def ispl():
    ensure_library()
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a GPU")
    import paper_2311_18737_amd as pkg

    return pkg


class Lines:
    """+-1 codes, unit noise, and in every 16th gate an echo with one line at a
    random frequency and random phases; gates step by L / 8, so echoes do not meet."""

    def __init__(self, L, N, G, P, snr_db, seed, sample_type="c64"):
        rng = np.random.default_rng(seed)
        step = max(1, L // 8)
        self.stride = (G - 1) * step + L
        self.geo = dict(code_len=L, fft_len=N, n_gates=G, gate_step=step, pulse_stride=self.stride,
                        sample_type=sample_type)
        self.tx = (rng.integers(0, 2, (P, L)) * 2 - 1).astype(np.complex64)
        x = rng.standard_normal((P, self.stride, 2), dtype=np.float32).view(np.complex64)[..., 0]
        x *= np.float32(np.sqrt(0.5))
        self.gates = list(range(3, G, 16))
        n = np.arange(L)
        amp = 10.0 ** (snr_db / 20.0)
        for g in self.gates:
            tone = amp * np.exp(2j * np.pi * rng.uniform() * n)
            phase = np.exp(2j * np.pi * rng.uniform(size=(P, 1)))
            x[:, g * step:g * step + L] += (self.tx * tone * phase).astype(np.complex64)
        if sample_type == "ci16":
            x = np.round(x.view(np.float32).reshape(P, self.stride, 2) * (2000.0 / max(1.0, amp)))
            x = x.astype(np.int16)
        self.x = x
        self.ref = oracle_spectra(self.x, self.tx, n_gates=G, gate_step=step, first_gate=0,
                                  fft_len=N, tx_per_pulse=True, gates=self.gates)

    def run(self, ispl):
        ctx = ispl.Context(max_pulses=len(self.tx), **self.geo)
        out = ctx.integrate_spectra(torch.from_numpy(self.x).to(DEV), torch.from_numpy(self.tx).to(DEV))
        got = out[self.gates].cpu().numpy().astype(np.float64)
        ctx.close()
        return got


SHAPES = [
    # L,   N,     G,   P
    (64, 4096, 600, 100),
    (256, 16384, 300, 100),
    (333, 8192, 300, 60),
    (1000, 16384, 200, 100),
    (2000, 32768, 120, 100),
    (4000, 16384, 100, 60),
    (8000, 32768, 60, 60),
]


@pytest.mark.parametrize("sample_type", ["c64", "ci16"])
@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: "L{}_N{}_G{}_P{}".format(*s))
def test_line_below_the_noise(ispl, shape, sample_type):
    """-10 dB per sample.  Bound: ten roundings of an FP32 transform (2^-24 each) as without a
    line, and a sixth of a rounding of the line's points, which its neighbours see."""
    L, N, G, P = shape
    lines = Lines(L, N, G, P, -10.0, seed=L, sample_type=sample_type)
    got, ref = lines.run(ispl), lines.ref
    mean = ref.mean(axis=1, keepdims=True)
    err = (np.abs(got - ref) / np.maximum(ref, mean)).max(axis=1)
    bound = 2.0 ** -24 * (10.0 + ref.max(axis=1) / mean[:, 0] / 6.0)
    assert (err <= bound).all(), (err / bound).max()


@pytest.mark.parametrize("sample_type", ["c64", "ci16"])
@pytest.mark.parametrize("snr_db", [0.0, 10.0, 20.0, 40.0])
@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: "L{}_N{}_G{}_P{}".format(*s))
def test_line_above_the_noise(ispl, shape, snr_db, sample_type):
    """Bins of power S are off by no more than an FP32 transform's rounding, d = 2^-25 x 64 of the
    gate's mean amplitude (4 deviations of 16 passes of two roundings), however strong the line: 2 d
    sqrt(S mean S) + d^2 mean S."""
    L, N, G, P = shape
    lines = Lines(L, N, G, P, snr_db, seed=L + 1, sample_type=sample_type)
    got, ref = lines.run(ispl), lines.ref
    mean = ref.mean(axis=1, keepdims=True)
    d = 2.0 ** -25 * 64.0
    bound = 2.0 * d * np.sqrt(ref * np.maximum(ref, mean)) + d * d * mean
    err = np.abs(got - ref) / bound
    assert err.max() <= 1.0, err.max()


@pytest.mark.parametrize("precision", ["fp16x3", "bf16x3"])
@pytest.mark.parametrize("snr_db", [-10.0, 0.0, 20.0, 40.0])
@pytest.mark.parametrize("shape", [s for s in SHAPES if s[0] <= 1000],
                         ids=lambda s: "L{}_N{}_G{}_P{}".format(*s))
def test_zoom_windows_of_lines(ispl, shape, snr_db, precision):
    """Windows at, beside and far from a line, as exact as split products: d = 8 x 2^-22 or 8 x 2^-16
    of the gate's mean amplitude."""
    L, N, G, P = shape
    K = 256
    lines = Lines(L, N, G, P, snr_db, seed=L + 2)
    ref = lines.ref
    start = np.zeros(G, dtype=np.int32)
    for i, g in enumerate(lines.gates):
        start[g] = int(ref[i].argmax()) - (128, 128, 2 * K, N // 2)[i % 4]
    ctx = ispl.Context(max_pulses=P, **lines.geo)
    zoom = ispl.Zoom(ctx, K, precision)
    out = zoom.spectra(torch.from_numpy(lines.x).to(DEV), torch.from_numpy(lines.tx).to(DEV),
                       torch.from_numpy(start).to(DEV))
    got = out[lines.gates].cpu().numpy().astype(np.float64)
    zoom.close()
    ctx.close()
    idx = (start[lines.gates].astype(np.int64)[:, None] + np.arange(K)) % N
    mean = ref.mean(axis=1, keepdims=True)
    want = np.take_along_axis(ref, idx, axis=1)
    d = 8.0 * 2.0 ** (-22 if precision == "fp16x3" else -16)
    bound = 2.0 * d * np.sqrt(want * np.maximum(want, mean)) + d * d * mean
    err = np.abs(got - want) / bound
    assert err.max() <= 1.0, err.max()


@pytest.mark.parametrize("shape", [(256, 16384, 300, 100), (1000, 16384, 200, 64)],
                         ids=lambda s: "L{}_N{}_G{}_P{}".format(*s))
def test_power_far_below_the_mean(ispl, shape):
    """Noise filtered to a fifth of the band (after decoding): the stop band, 60 dB down, keeps the
    accuracy of an FP32 transform."""
    L, N, G, P = shape
    rng = np.random.default_rng(L)
    step = L
    stride = G * step
    tx = (rng.integers(0, 2, (P, L)) * 2 - 1).astype(np.complex64)
    taper = np.blackman(L)
    f = np.fft.fftfreq(L)
    keep = np.abs(f) < 0.1
    y = np.empty((P, G, L), dtype=np.complex64)
    for p in range(P):
        z = (rng.standard_normal((G, L)) + 1j * rng.standard_normal((G, L))) * np.where(keep, 1.0, 1e-3)
        y[p] = np.fft.ifft(z, axis=1) * taper * np.sqrt(L)
    x = (y * tx[:, None, :]).reshape(P, stride)
    gates = list(range(0, G, 37))
    ref = oracle_spectra(x, tx, n_gates=G, gate_step=step, first_gate=0, fft_len=N, tx_per_pulse=True,
                         gates=gates)
    ctx = ispl.Context(code_len=L, fft_len=N, n_gates=G, gate_step=step, pulse_stride=stride,
                       max_pulses=P)
    out = ctx.integrate_spectra(torch.from_numpy(x).to(DEV), torch.from_numpy(tx).to(DEV))
    got = out[gates].cpu().numpy().astype(np.float64)
    ctx.close()
    mean = ref.mean(axis=1, keepdims=True)
    assert (ref < 1e-4 * mean).any()
    d = 2.0 ** -25 * 64.0
    bound = 2.0 * d * np.sqrt(ref * np.maximum(ref, mean)) + d * d * mean
    assert (np.abs(got - ref) / bound).max() <= 1.0


@pytest.mark.parametrize("when", ["always", "late", "early"])
@pytest.mark.parametrize("case", [
    # L,    N,     G,   P,   type, per-pulse codes
    (1000, 16384, 400, 200, "c64", True),
    (1000, 16384, 400, 201, "ci16", False),
    (300, 8192, 900, 333, "ci16", True),
    (4000, 16384, 260, 130, "ci16", True),
    (2000, 32768, 300, 129, "c64", False),
    (6000, 32768, 130, 100, "c64", True),
], ids=lambda c: "L{}_N{}_G{}_P{}_{}_{}".format(*c))
def test_long_calls_of_mixed_gates(ispl, case, when):
    """Calls long enough that gates with strong lines are looked for after their first pulses: lines
    of 5 to 30 dB in some gates, in all pulses, only in the last half or only in the first tenth;
    every tested gate, with and without a line, as exact as by an FP32 transform.  Listed gates and
    accumulation give the same rows."""
    L, N, G, P, st, per = case
    rng = np.random.default_rng(L + P)
    step = max(1, L // 8)
    stride = 5 + (G - 1) * step + L
    tx = (rng.integers(0, 2, (P if per else 1, L)) * 2 - 1).astype(np.complex64)
    x = rng.standard_normal((P, stride, 2), dtype=np.float32).view(np.complex64)[..., 0]
    x *= np.float32(np.sqrt(0.5))
    pulses = {"always": slice(0, P), "late": slice(P // 2, P), "early": slice(0, P // 10)}[when]
    n = np.arange(L)
    hot = list(range(7, G, 40))
    for i, g in enumerate(hot):
        tone = 10.0 ** ((5.0 + 25.0 * i / len(hot)) / 20.0) * np.exp(2j * np.pi * rng.uniform() * n)
        at = 5 + g * step
        x[pulses, at:at + L] += (tx[pulses] if per else tx) * tone.astype(np.complex64)
    if st == "ci16":
        x = np.round(x.view(np.float32).reshape(P, stride, 2) * 200.0).astype(np.int16)
    gates = sorted(hot[:6] + [g + 20 for g in hot[:6] if g + 20 < G])
    ref = oracle_spectra(x, tx, n_gates=G, gate_step=step, first_gate=5, fft_len=N, tx_per_pulse=per,
                         gates=gates)
    ctx = ispl.Context(code_len=L, fft_len=N, n_gates=G, gate_step=step, first_gate=5,
                       pulse_stride=stride, sample_type=st, max_pulses=P)
    xs, xt = torch.from_numpy(x).to(DEV), torch.from_numpy(tx).to(DEV)
    out = ctx.integrate_spectra(xs, xt)
    got = out[gates].cpu().numpy().astype(np.float64)
    mean = ref.mean(axis=1, keepdims=True)
    d = 2.0 ** -25 * 64.0
    bound = 2.0 * d * np.sqrt(ref * np.maximum(ref, mean)) + d * d * mean
    assert (np.abs(got - ref) / bound).max() <= 1.0
    again = ctx.integrate_spectra(xs, xt, out=out.clone(), accumulate=True)
    np.testing.assert_allclose(again.cpu().numpy(), 2 * out.cpu().numpy(), rtol=1e-6)
    lst = torch.tensor(gates[::-1], dtype=torch.int32, device=DEV)
    part = torch.full((G, N), -1.0, device=DEV)
    lst = torch.cat([lst, torch.zeros(G - len(gates), dtype=torch.int32, device=DEV)])
    ctx.integrate_spectra(xs, xt, out=part,
                          gates=(lst, torch.tensor([len(gates)], dtype=torch.int32, device=DEV)))
    listed = part[gates].cpu().numpy().astype(np.float64)
    assert (np.abs(listed - ref) / bound).max() <= 1.0
    rest = torch.ones(G, dtype=torch.bool, device=DEV)
    rest[gates] = False
    assert bool((part[rest] == -1.0).all())
    ctx.close()


@pytest.mark.parametrize("case", [
    # L,   N,    G,  P,  K,   type, per-pulse codes
    (100, 4096, 24, 20, 128, "c64", True),
    (256, 16384, 40, 60, 256, "c64", False),
    (130, 2048, 70, 33, 384, "c64", True),
    (2000, 16384, 9, 25, 128, "c64", True),
], ids=lambda c: "L{}_N{}_G{}_P{}_K{}_{}_{}".format(*c))
def test_zoom_of_gates_far_apart_in_power(ispl, case):
    """Gates from 0 to -160 dB side by side in every pulse: each one's window keeps the FP16 split's
    accuracy relative to its own mean."""
    L, N, G, P, K, st, per = case
    rng = np.random.default_rng(L)
    stride = G * L
    tx = (rng.integers(0, 2, (P if per else 1, L)) * 2 - 1).astype(np.complex64)
    scale = 10.0 ** (-8.0 * rng.permutation(G) / (G - 1))
    x = rng.standard_normal((P, G, L, 2)).view(np.complex128)[..., 0] * scale[None, :, None]
    x = x.reshape(P, stride).astype(np.complex64)
    ref = oracle_spectra(x, tx, n_gates=G, gate_step=L, first_gate=0, fft_len=N, tx_per_pulse=per)
    start = rng.integers(0, N, G).astype(np.int32)
    ctx = ispl.Context(code_len=L, fft_len=N, n_gates=G, gate_step=L, pulse_stride=stride,
                       sample_type=st, max_pulses=P)
    zoom = ispl.Zoom(ctx, K, "fp16x3")
    out = zoom.spectra(torch.from_numpy(x).to(DEV), torch.from_numpy(tx).to(DEV),
                       torch.from_numpy(start).to(DEV))
    got = out.cpu().numpy().astype(np.float64)
    zoom.close()
    ctx.close()
    idx = (start.astype(np.int64)[:, None] + np.arange(K)) % N
    mean = ref.mean(axis=1, keepdims=True)
    want = np.take_along_axis(ref, idx, axis=1)
    d = 8.0 * 2.0 ** -22
    bound = 2.0 * d * np.sqrt(want * np.maximum(want, mean)) + d * d * mean
    assert (np.abs(got - want) / bound).max() <= 1.0


@pytest.mark.parametrize("sample_type", ["c64", "ci16"])
def test_lines_in_every_slice(ispl, sample_type):
    """More gates than the grid scratch holds, in calls that look for lines early: lines of 15 dB in
    gates of the first and the last slice, in whole calls and in listed ones."""
    L, N, G, P, step = 3000, 16384, 2200, 130, 2
    rng = np.random.default_rng(7)
    stride = (G - 1) * step + L
    tx = (rng.integers(0, 2, (P, L)) * 2 - 1).astype(np.complex64)
    x = rng.standard_normal((P, stride, 2), dtype=np.float32).view(np.complex64)[..., 0]
    hot = [5, 1090, 1110, 2190]
    n = np.arange(L)
    for g in hot:
        tone = 10.0 ** (15.0 / 20.0) * np.exp(2j * np.pi * rng.uniform() * n)
        x[:, g * step:g * step + L] += (tx * tone).astype(np.complex64)
    if sample_type == "ci16":
        x = np.round(x.view(np.float32).reshape(P, stride, 2) * 200.0).astype(np.int16)
    gates = sorted(hot + [0, 6, 1099, 1100, 1101, 2199])
    ref = oracle_spectra(x, tx, n_gates=G, gate_step=step, first_gate=0, fft_len=N, tx_per_pulse=True,
                         gates=gates)
    mean = ref.mean(axis=1, keepdims=True)
    d = 2.0 ** -25 * 64.0
    bound = 2.0 * d * np.sqrt(ref * np.maximum(ref, mean)) + d * d * mean
    ctx = ispl.Context(code_len=L, fft_len=N, n_gates=G, gate_step=step, pulse_stride=stride,
                       sample_type=sample_type, max_pulses=P)
    xs, xt = torch.from_numpy(x).to(DEV), torch.from_numpy(tx).to(DEV)
    out = ctx.integrate_spectra(xs, xt)
    got = out[gates].cpu().numpy().astype(np.float64)
    assert (np.abs(got - ref) / bound).max() <= 1.0
    # the tested gates last in a list of most
    order = np.concatenate([np.setdiff1d(np.arange(0, G, 1), gates)[: G - 100], gates]).astype(np.int32)
    lst = torch.zeros(G, dtype=torch.int32, device=DEV)
    lst[:len(order)] = torch.from_numpy(order).to(DEV)
    count = torch.tensor([len(order)], dtype=torch.int32, device=DEV)
    part = torch.zeros_like(out)
    ctx.integrate_spectra(xs, xt, out=part, gates=(lst, count))
    got = part[gates].cpu().numpy().astype(np.float64)
    rest = np.setdiff1d(np.arange(G), order)
    ctx.close()
    assert (np.abs(got - ref) / bound).max() <= 1.0
    assert not part[rest.tolist()].any()


@pytest.mark.parametrize("case", [
    # L,   N,     G,   P,   K,   type, per-pulse codes
    (256, 16384, 1000, 400, 256, "c64", True),
    (700, 8192, 400, 301, 128, "ci16", False),
], ids=lambda c: "L{}_N{}_G{}_P{}_K{}_{}_{}".format(*c))
def test_zoom_of_long_calls_of_mixed_gates(ispl, case):
    """Windows of calls that look for lines early: lines of 30 dB in some gates, all calls and listed
    ones, at the FP16 split's accuracy."""
    L, N, G, P, K, st, per = case
    rng = np.random.default_rng(L + G)
    step, hot = 3, [2, G // 2, G - 1]
    stride = (G - 1) * step + L
    tx = (rng.integers(0, 2, (P if per else 1, L)) * 2 - 1).astype(np.complex64)
    x = rng.standard_normal((P, stride, 2), dtype=np.float32).view(np.complex64)[..., 0]
    freq = rng.uniform(size=G)
    for g in hot:
        tone = 10.0 ** (30.0 / 20.0) * np.exp(2j * np.pi * freq[g] * np.arange(L))
        x[:, g * step:g * step + L] += (tx * tone).astype(np.complex64)
    if st == "ci16":
        x = np.round(x.view(np.float32).reshape(P, stride, 2) * 100.0).astype(np.int16)
    start = (np.round(freq * N).astype(np.int64) - K // 2).astype(np.int32)
    gates = sorted(hot + [0, 1, 3, G // 2 + 1, G - 2])
    ref = oracle_spectra(x, tx, n_gates=G, gate_step=step, first_gate=0, fft_len=N, tx_per_pulse=per,
                         gates=gates)
    mean = ref.mean(axis=1, keepdims=True)
    want = np.take_along_axis(ref, (start[gates].astype(np.int64)[:, None] + np.arange(K)) % N, axis=1)
    d = 8.0 * 2.0 ** -22
    bound = 2.0 * d * np.sqrt(want * np.maximum(want, mean)) + d * d * mean
    ctx = ispl.Context(code_len=L, fft_len=N, n_gates=G, gate_step=step, pulse_stride=stride,
                       sample_type=st, max_pulses=P)
    zoom = ispl.Zoom(ctx, K, "fp16x3")
    args = (torch.from_numpy(x).to(DEV), torch.from_numpy(tx).to(DEV), torch.from_numpy(start).to(DEV))
    out = zoom.spectra(*args)
    got = out[gates].cpu().numpy().astype(np.float64)
    lst = torch.zeros(G, dtype=torch.int32, device=DEV)
    lst[:len(gates)] = torch.tensor(gates[::-1], dtype=torch.int32, device=DEV)
    count = torch.tensor([len(gates)], dtype=torch.int32, device=DEV)
    part = torch.full_like(out, -1.0)
    zoom.spectra(*args, out=part, gates=(lst, count))
    listed = part[gates].cpu().numpy().astype(np.float64)
    rest = torch.ones(G, dtype=torch.bool, device=DEV)
    rest[gates] = False
    assert bool((part[rest] == -1.0).all())
    zoom.close()
    ctx.close()
    assert (np.abs(got - want) / bound).max() <= 1.0
    assert (np.abs(listed - want) / bound).max() <= 1.0
