"""The matrix-product zoom at lengths that no grid serves (2 L - 1 > N, or L > 1024), where every
call runs it: sign-bit and complex codes, several pulse blocks and chunks, ragged tails, listed
gates, accumulation.  Against the FP64 oracle; the tolerances are those of the split products
(FP16 1e-5, BF16 2e-4, relative to max(bin, gate mean))."""

import numpy as np
import pytest

torch = pytest.importorskip("torch")

from oracle import window_spectra  # noqa: E402
from synth import random_inputs  # noqa: E402
from tests.conftest import ensure_library  # noqa: E402
from tests.parity_util import spectra_error  # noqa: E402

pytestmark = pytest.mark.gpu

DEV = "cuda:0"
TOL = {"fp16x3": 1e-5, "bf16x3": 2e-4}


@pytest.fixture(scope="module")
def ispl():
    ensure_library()
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a GPU")
    import paper_2311_18737_amd as pkg

    return pkg


SHAPES = [
    # N, L, G, P, s, g0, type, per-pulse, kind, K
    # two pulse chunks of three 64-pulse blocks each, the last partial; a ragged last chunk of samples
    (1024, 600, 256, 300, 1, 0, "c64", True, "bpsk", 128),
    (1024, 900, 300, 200, 2, 0, "ci16", True, "bpsk", 256),
    # the same with one code for all pulses, and with complex ones
    (1024, 600, 256, 130, 1, 0, "ci16", False, "bpsk", 128),
    (1024, 600, 256, 300, 1, 0, "ci16", True, "phase", 256),
    # one 32-pulse block per chunk (FP16 exponents of each gate), L not a multiple of 4
    (1024, 515, 40, 130, 3, 2, "c64", True, "bpsk", 256),
    (1024, 513, 9, 1, 7, 1, "ci16", True, "gauss", 1024),
    # 33 pulses: one of the second column tile
    (16384, 1025, 5, 33, 11, 0, "ci16", True, "bpsk", 640),
    # exponents of each gate: one gate of the last eight
    (16384, 1030, 17, 65, 5, 0, "c64", False, "bpsk", 128),
    # no sample twiddles in LDS, sign bits
    (16384, 4100, 3, 70, 25, 3, "c64", True, "bpsk", 384),
]


def run(ispl, case, precision, samples, tx, starts, **kw):
    N, L, G, P, s, g0, st, per, kind, K = case
    ctx = ispl.Context(code_len=L, fft_len=N, n_gates=G, gate_step=s, first_gate=g0,
                       pulse_stride=samples.shape[1], sample_type=st, max_pulses=P)
    zoom = ispl.Zoom(ctx, K, precision)
    out = zoom.spectra(torch.from_numpy(samples).to(DEV), torch.from_numpy(tx).to(DEV),
                       torch.from_numpy(starts.astype(np.int32)).to(DEV), **kw)
    got = out.cpu().numpy()
    zoom.close()
    ctx.close()
    return got


def inputs(case):
    N, L, G, P, s, g0, st, per, kind, K = case
    print(f"case {case}", flush=True)
    samples, tx = random_inputs(P, g0 + (G - 1) * s + L + 3, L, sample_type=st, code_kind=kind,
                                tx_rows=None if per else 1, seed=N + L + K,
                                amplitude=3000.0 if st == "ci16" else 1.0)
    return samples, tx, np.random.default_rng(L + P).integers(-2 * N, 2 * N, size=G)


def reference(case, samples, tx, starts):
    N, L, G, P, s, g0, st, per, kind, K = case
    return window_spectra(samples, tx, n_gates=G, gate_step=s, first_gate=g0, fft_len=N,
                          tx_per_pulse=per, bin_start=starts, n_bins=K)


@pytest.mark.parametrize("case", SHAPES, ids=lambda t: "N{}_L{}_G{}_P{}_{}_{}_{}_K{}".format(
    *t[:4], *t[6:9], t[9]))
def test_products_match_oracle(ispl, case):
    samples, tx, starts = inputs(case)
    ref = reference(case, samples, tx, starts)
    for precision in ("fp16x3", "bf16x3"):
        err = spectra_error(run(ispl, case, precision, samples, tx, starts), ref)
        assert err["max_e"] <= TOL[precision], (precision, err)


@pytest.mark.parametrize("pulse", [0, 70, 99])
def test_sign_bits_beside_a_complex_row(ispl, pulse):
    """One complex chip sends its pulse chunk (0..49 or 50..99) to the complex codes; the other
    stays on sign bits."""
    case = (1024, 520, 300, 100, 2, 0, "c64", True, "bpsk", 256)
    samples, tx, starts = inputs(case)
    tx[pulse, 3] = np.exp(0.3j)
    ref = reference(case, samples, tx, starts)
    for precision in ("fp16x3", "bf16x3"):
        err = spectra_error(run(ispl, case, precision, samples, tx, starts), ref)
        assert err["max_e"] <= TOL[precision], (precision, err)


@pytest.mark.parametrize("case", [
    (1024, 600, 70, 300, 1, 0, "ci16", True, "bpsk", 128),   # FP16 exponents of each pulse, chunks
    (16384, 1027, 40, 50, 3, 1, "c64", False, "phase", 256),  # of each pulse and gate
], ids=lambda t: "L{}_G{}_P{}".format(t[1], t[2], t[3]))
@pytest.mark.parametrize("listed", [0, 1, 33])
def test_listed_gates(ispl, case, listed):
    """Listed gates get the whole call's rows bit for bit, added to what is there; the others stay."""
    samples, tx, starts = inputs(case)
    G, K = case[2], case[9]
    order = np.random.default_rng(listed).permutation(G).astype(np.int32)
    for precision in ("fp16x3", "bf16x3"):
        full = run(ispl, case, precision, samples, tx, starts)
        out = torch.full((G, K), 7.0, device=DEV)
        gates = (torch.from_numpy(order).to(DEV), torch.tensor([listed], dtype=torch.int32, device=DEV))
        got = run(ispl, case, precision, samples, tx, starts, out=out, accumulate=True, gates=gates)
        want = np.full((G, K), 7.0, dtype=np.float32)
        want[order[:listed]] += full[order[:listed]]
        assert np.array_equal(got, want), precision
