"""The key switch of gate levels at every build of its int8 GEMM (one to four
slot blocks per input coefficient, base 2 among them) and with both workgroup
shapes: MUX gates add a second ciphertext, gates without a bootstrap or with an
invalid wire have none.  Every wire equals the oracle's."""
import concurrent.futures as cf
import os
import sys

import numpy as np
import pytest

import test_gpu_keyswitch as K
from paper_2306_11006_amd import inputs

pytestmark = pytest.mark.gpu

THREADS = min(16, os.cpu_count() or 4)


@pytest.mark.parametrize("p", K.SETS, ids=[p.name for p in K.SETS])
def test_level_key_switch_bit_exact(O, p):
    import dataclasses
    from paper_2306_11006_amd import cggi
    p = dataclasses.replace(p, n=min(p.n, 40))
    seed = 9800 + p.ks_base_bit * 100 + p.ks_t
    bsk, ksk = inputs.uniform_keys(p, seed)
    ctx = cggi.Context(p, cggi.to_device(bsk), cggi.to_device(ksk),
                       forms=("ntt",))
    for G in (3, 47, 49, 130):
        g = inputs.rng(seed + G).integers(0, 20, size=(G, 5))
        g[:, 0] = np.arange(G) % 11
        g[:, 4] = 20 + np.arange(G)
        g = g.astype(np.int32)
        wires = inputs.uniform_lwe(p, seed + 1, 20 + G)
        bad = G // 2
        g[bad, 1] = 10**6                       # skipped: its wire stays
        with cf.ThreadPoolExecutor(THREADS) as ex:
            want = np.stack(list(ex.map(
                lambda t: wires[t[4]] if t[4] == 20 + bad else
                O.gate(p, int(t[0]), bsk, ksk, wires[t[1]], wires[t[2]],
                       wires[t[3]]), g)))
        print(f"level key switch {p.name} G={G}", file=sys.stderr, flush=True)
        w = cggi.to_device(wires)
        ctx.eval_level("ntt", cggi.to_device(g), w)
        assert np.array_equal(cggi.to_host(w)[20:], want), G
    ctx.close()
