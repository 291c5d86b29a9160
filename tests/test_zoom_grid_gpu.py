"""Zoom windows from the pulse-summed grid: code lengths on both sides of every
grid length, windows of one to many 128-bin runs (split over workgroups or not),
window starts that wrap or are negative, gate lists, accumulation, more gates than
the scratch holds, and powers beyond the FP32 range, against the FP64 oracle.

Tolerance: the plain path's 1e-5 of max(S, mean S) per bin (parity_util): the pulses
are summed in FP32, the windows expanded in FP64."""

import numpy as np
import pytest

torch = pytest.importorskip("torch")

from oracle import integrate_spectra as oracle_spectra  # noqa: E402
from synth import random_inputs  # noqa: E402
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


def window(ref, starts, K):
    N = ref.shape[1]
    idx = (np.asarray(starts)[:, None] + np.arange(K)) % N
    return np.take_along_axis(ref, idx, axis=1)


def check(got, ref, starts, K, gates=None):
    want = window(ref, starts, K)
    scale = np.maximum(want, ref.mean(axis=1, keepdims=True))
    err = np.abs(got - want) / scale
    assert err.max() <= 1e-5, err.max()


CASES = [
    # N,    L,    G,  P, K,    type,  per-pulse, kind
    (1024, 1, 2, 5, 128, "c64", True, "phase"),
    (1024, 64, 3, 9, 1024, "ci16", True, "bpsk"),
    (1024, 65, 3, 2, 256, "c64", False, "gauss"),
    (1024, 512, 4, 7, 384, "c64", True, "bpsk"),
    (2048, 513, 3, 4, 128, "ci16", True, "phase"),
    (2048, 1024, 2, 3, 2048, "c64", True, "gauss"),
    (4096, 129, 70, 520, 256, "ci16", True, "bpsk"),
    (16384, 256, 5, 1, 640, "c64", True, "bpsk"),
    (16384, 257, 300, 6, 256, "c64", False, "bpsk"),
    (65536, 1000, 2, 3, 4096, "c64", True, "phase"),
    (65536, 2, 600, 4, 128, "ci16", True, "bpsk"),
]


@pytest.mark.parametrize("case", CASES, ids=lambda t: "N{}_L{}_G{}_P{}_K{}_{}_{}_{}".format(*t))
def test_windows_match_oracle(ispl, case):
    N, L, G, P, K, st, per, kind = case
    s = max(1, L // 3)
    stride = (G - 1) * s + L + 1
    samples, tx = random_inputs(P, stride, L, sample_type=st, code_kind=kind,
                                tx_rows=None if per else 1, seed=N + L,
                                amplitude=3000.0 if st == "ci16" else 1.0)
    ref = oracle_spectra(samples, tx, n_gates=G, gate_step=s, first_gate=1, fft_len=N,
                         tx_per_pulse=per)
    rng = np.random.default_rng(L)
    starts = rng.integers(-N, 2 * N, G).astype(np.int32)
    starts[0] = N - 1
    ctx = ispl.Context(code_len=L, fft_len=N, n_gates=G, gate_step=s, first_gate=1,
                       pulse_stride=stride, sample_type=st, max_pulses=P)
    zoom = ispl.Zoom(ctx, K, "fp16x3")
    xs, xt = torch.from_numpy(samples).to(DEV), torch.from_numpy(tx).to(DEV)
    k0 = torch.from_numpy(starts).to(DEV)
    out = zoom.spectra(xs, xt, k0)
    torch.cuda.synchronize()
    check(out.cpu().numpy(), ref, starts, K)
    # a second call adds to the first, up to the rounding of the sum
    twice = zoom.spectra(xs, xt, k0, out=out.clone(), accumulate=True)
    torch.cuda.synchronize()
    assert torch.equal(twice, out + out)
    # listed gates are the full call's rows, the others untouched
    lst = torch.arange(G - 1, -1, -1, dtype=torch.int32, device=DEV)
    part = torch.full((G, K), -1.0, device=DEV)
    n = (G + 1) // 2
    zoom.spectra(xs, xt, k0, out=part,
                 gates=(lst, torch.tensor([n], dtype=torch.int32, device=DEV)))
    torch.cuda.synchronize()
    assert torch.equal(part[G - n:], out[G - n:]) and bool((part[:G - n] == -1.0).all())
    zoom.close()
    ctx.close()


@pytest.mark.parametrize("L,N", [(100, 2048), (700, 16384)])
def test_powers_beyond_fp32_and_nan(ispl, L, N):
    G, P, K = 5, 4, N
    stride = G * L
    samples, tx = random_inputs(P, stride, L, code_kind="bpsk", seed=9)
    tone = np.exp(2j * np.pi * 0.125 * np.arange(L))
    samples[:, L:2 * L] = samples[:, L:2 * L] * 1e16 + 3e18 * tx * tone  # gate 1: overflows
    samples[:, 2 * L:3 * L] *= 1e-18                                     # gate 2: tiny powers
    samples[:, 3 * L:4 * L] = 0                                          # gate 3: no echo
    samples[2, 4 * L + 5] = np.nan                                       # gate 4
    ctx = ispl.Context(code_len=L, fft_len=N, n_gates=G, gate_step=L, pulse_stride=stride,
                       max_pulses=P)
    zoom = ispl.Zoom(ctx, K, "fp16x3")
    starts = np.zeros(G, dtype=np.int32)
    out = zoom.spectra(torch.from_numpy(samples).to(DEV), torch.from_numpy(tx).to(DEV),
                       torch.from_numpy(starts).to(DEV))
    torch.cuda.synchronize()
    got = out.cpu().numpy().astype(np.float64)
    with np.errstate(all="ignore"):
        ref = oracle_spectra(samples, tx, n_gates=G, gate_step=L, first_gate=0, fft_len=N,
                             tx_per_pulse=True)
    big = float(np.finfo(np.float32).max)
    over, under = ref[1] > 1.0001 * big, ref[1] < 0.9999 * big
    assert over.any() and under.any()
    assert np.isinf(got[1][over]).all() and np.isfinite(got[1][under]).all()
    for g in (0, 2):
        check(got[g:g + 1], ref[g:g + 1], starts[:1], K)
    assert (got[3] == 0).all() and np.isnan(got[4]).all()
    zoom.close()
    ctx.close()
