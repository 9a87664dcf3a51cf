"""The double-precision transform kernel at the edges of its range: every ring
degree, digit counts with and without a compile-time build, the widest digits
its error bound admits, batches around a CU's and the chip's width, and keys
and test vectors at the extremes of their halves (the sums and so the rounding
errors at their largest); and the modular transform kernel past the bound,
where it still serves.  Tolerance 0 against the oracle: the results are
integers."""
import concurrent.futures as cf
import os
import sys

import numpy as np
import pytest

from paper_2306_11006_amd import inputs, params

pytestmark = pytest.mark.gpu

THREADS = min(16, os.cpu_count() or 4)


def case(n, N, bg, l):
    return params.Params(f"n{n}_N{N}_bg{bg}_l{l}", n=n, N=N, k=1, bg_bit=bg,
                         l=l, ks_base_bit=2, ks_t=4, lwe_noise_log2=15,
                         bk_noise_log2=25)


def bound(p):
    M, m, R = p.N // 2, (p.N // 2).bit_length() - 1, 2 * p.l
    return (2 * R * M ** 1.5 * 2.0 ** (p.bg_bit - 1) * 2.0 ** 15 *
            (15 * m + 2 * 2 ** 0.5 * R) * 2.0 ** -53)


# within the bound: the widest digits per ring, then l = 1 .. 5 with odd step
# counts around the 64 rotations a wave holds
INSIDE = [case(65, 256, 16, 1), case(3, 512, 14, 2), case(64, 1024, 14, 1),
          case(5, 2048, 11, 2), case(63, 256, 7, 3), case(130, 512, 10, 3),
          case(33, 1024, 10, 2), case(1, 1024, 7, 3), case(20, 1024, 7, 4),
          case(9, 2048, 7, 3), case(7, 2048, 9, 1), case(6, 256, 6, 5)]
# past it: the modular transform kernel
PAST = [case(20, 256, 18, 1), case(9, 512, 17, 1), case(12, 1024, 16, 1),
        case(5, 2048, 15, 2)]


def check(O, p, forms, seed, B, extreme):
    import torch
    from paper_2306_11006_amd import cggi
    bsk, ksk = inputs.uniform_keys(p, seed)
    cts = inputs.uniform_lwe(p, seed + 1, B)
    testv = None
    if extreme:
        # halves at -2^15 / 2^15 - 1 in runs, alternating accumulators
        g = inputs.rng(seed + 2)
        bsk = np.where(g.integers(0, 2, size=bsk.shape) == 1,
                       np.uint32(0x7FFF7FFF), np.uint32(0x80008000))
        bsk[:, :, 0] = np.uint32(0x7FFF8000)
        testv = np.where(np.arange(p.N) % 3 == 0, np.uint32(0x80000000),
                         np.uint32(0x7FFFFFFF)).astype(np.uint32)
    with cf.ThreadPoolExecutor(THREADS) as ex:
        want = np.stack(list(ex.map(
            lambda x: O.bootstrap(p, bsk, x) if testv is None
            else O.bootstrap(p, bsk, x, testv), cts)))
    ctx = cggi.Context(p, cggi.to_device(bsk), cggi.to_device(ksk),
                       forms=forms)
    tv = None if testv is None else cggi.to_device(testv)
    for form in forms:
        print(f"fft {p.name} form={form} B={B} extreme={extreme}",
              file=sys.stderr, flush=True)
        out = ctx.bootstrap(form, cggi.to_device(cts), testv=tv)
        torch.cuda.synchronize()
        assert np.array_equal(cggi.to_host(out), want), (p.name, form)
    ctx.close()


@pytest.mark.parametrize("extreme", [False, True], ids=["uniform", "extreme"])
@pytest.mark.parametrize("p", INSIDE, ids=[p.name for p in INSIDE])
def test_transform_kernel_bit_exact(O, p, extreme):
    assert bound(p) <= 0.25
    # the int8 form refuses many of these sets (digit operands past the LDS)
    forms = ("ntt", "int8") if p.bg_bit <= 7 and p.l <= 3 else ("ntt",)
    check(O, p, forms, 9100 + INSIDE.index(p), 5, extreme)


@pytest.mark.parametrize("p", PAST, ids=[p.name for p in PAST])
def test_modular_kernel_serves_past_the_bound(O, p):
    assert bound(p) > 0.25
    check(O, p, ("ntt",), 9200 + PAST.index(p), 5, False)


@pytest.mark.parametrize("B", [1, 255, 257, 600])
def test_transform_kernel_batch_widths(O, B):
    check(O, case(4, 1024, 7, 3), ("int8",), 9300 + B, B, False)
