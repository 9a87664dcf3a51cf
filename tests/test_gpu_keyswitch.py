"""The int8-GEMM key switch at the edges of its dispatch: one to four slot
blocks per input coefficient (each build of the kernel, base 2 among them),
batches around the row tiles and the change of workgroup shape, and column
counts that leave waves without a tile; every output equals the oracle's."""
import sys

import numpy as np
import pytest

from paper_2306_11006_amd import inputs, params

pytestmark = pytest.mark.gpu


def case(n, N, base, t):
    return params.Params(f"n{n}_N{N}_ks{base}x{t}", n=n, N=N, k=1, bg_bit=7,
                         l=2, ks_base_bit=base, ks_t=t, lwe_noise_log2=15,
                         bk_noise_log2=25)


# slot blocks of 32 per coefficient: 1, 2, 3, 4, and base 2 with 1 and 2
SETS = [case(31, 256, 2, 8), case(32, 512, 3, 5), case(70, 256, 3, 10),
        case(127, 256, 4, 7), case(5, 1024, 1, 9), case(40, 256, 1, 31)]


@pytest.mark.parametrize("p", SETS, ids=[p.name for p in SETS])
def test_key_switch_bit_exact(O, p):
    import torch
    from paper_2306_11006_amd import cggi
    seed = 9400 + SETS.index(p)
    bsk, ksk = inputs.uniform_keys(p, seed)
    big = inputs.uniform_lwe(p, seed + 1, 129, dim=p.N)
    want = np.stack([O.keyswitch(p, ksk, x) for x in big])
    ctx = cggi.Context(p, cggi.to_device(bsk), cggi.to_device(ksk),
                       forms=("ntt",))
    for B in (1, 32, 33, 48, 49, 64, 65, 128, 129):
        print(f"key switch {p.name} B={B}", file=sys.stderr, flush=True)
        out = ctx.keyswitch(cggi.to_device(big[:B]))
        torch.cuda.synchronize()
        assert np.array_equal(cggi.to_host(out), want[:B]), B
    ctx.close()
