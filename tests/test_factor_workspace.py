"""The f16-piece build's packed factor fits the memory it is given (host arithmetic only).

The packed L^-1 takes 12 bytes for each of N rows of N columns padded to 32, and the row
and column exponents 8 N more: for small N that are no multiple of 32 this is more than
the 16 N^2 bytes of the Gram it replaces."""
import numpy as np

from paper_2410_06129_amd import synth


def test_footprint_holds_the_packed_factor():
    """A plan that runs on f16 pieces pads W's rows to 32 columns, which its size shows
    beside the same plan on FP32 instructions (4M)."""
    from paper_2410_06129_amd import pinv as P
    on = []
    for N in list(range(1, 300)) + [352, 383, 384, 385]:
        M = int(2e9) // N ** 2 + N
        if M >= 1 << 27:
            continue
        C = -(-M // 4000) if M > 4000 else 1
        K = -(-M // C)
        enc = synth.Encoding(N, 1, np.zeros((K, 2)), t=None,
                             coil=np.ones((C, N), complex) if C > 1 else None)
        size = {c: P.pinv_encoding_key(enc, 1e-2, prec=P.FP32, cprod=c, flags=P.FLAG_UNCACHED)[1]
                for c in (P.CPROD_AUTO, P.CPROD_4M)}
        padded, plain = -(-N // 32) * 32, 16 * N * N
        factor = 12 * N * padded + 8 * N
        if size[P.CPROD_AUTO] == size[P.CPROD_4M]:
            assert N < 256 or N % 32 == 0, N          # FP32 tiles, or nothing to pad
            continue
        on.append(N)
        assert size[P.CPROD_AUTO] - size[P.CPROD_4M] == 8 * C * K * (padded - N) + max(0, factor - plain)
        assert factor <= plain, N                     # below this N the measurements do not reach
    assert on and min(on) > 256
