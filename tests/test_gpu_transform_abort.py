"""The latency-mode error word set while int8 batches of latency mode's widths
run on the transform kernel: a bootstrap then writes its whole output or
nothing, so every row equals the reference or is untouched, and the rows of
launches made after the abort are untouched."""
import sys

import numpy as np
import pytest

from paper_2306_11006_amd import inputs, params

pytestmark = pytest.mark.gpu

MARK = 0x5A5A5A5A


def test_abort_while_batches_run():
    import torch
    from paper_2306_11006_amd import cggi
    p = params.DEFAULT
    bsk, ksk = inputs.uniform_keys(p, 7700)
    ctx = cggi.Context(p, cggi.to_device(bsk), cggi.to_device(ksk))
    B = 64
    cts = cggi.to_device(inputs.uniform_lwe(p, 7701, B))
    ref = ctx.bootstrap("ntt", cts)
    outs = [torch.full((B, p.N + 1), MARK, dtype=torch.int32, device="cuda")
            for _ in range(12)]
    torch.cuda.synchronize()
    print(f"abort during {len(outs)} launches of {B}", file=sys.stderr,
          flush=True)
    for out in outs[:-1]:
        ctx.bootstrap("int8", cts, out)
    ctx.latency_abort()
    ctx.bootstrap("int8", cts, outs[-1])
    torch.cuda.synchronize()
    assert bool((outs[-1] == MARK).all())
    for k, out in enumerate(outs):
        right = (out == ref).all(dim=1)
        untouched = (out == MARK).all(dim=1)
        assert bool((right | untouched).all()), k
    with pytest.raises(cggi.CggiError) as e:
        ctx.check()
    assert e.value.code == cggi.E_TIMEOUT
    assert np.array_equal(cggi.to_host(ctx.bootstrap("int8", cts)),
                          cggi.to_host(ref))
    ctx.check()
    ctx.close()


def test_capture_after_an_abort_keeps_the_bootstraps():
    """A graph captured between an abort and the check replays the bootstraps
    (three replays, eager work between); an eager call there does nothing."""
    import torch
    from paper_2306_11006_amd import cggi
    p = params.TOY
    bsk, ksk = inputs.uniform_keys(p, 7710)
    ctx = cggi.Context(p, cggi.to_device(bsk), cggi.to_device(ksk))
    cts = cggi.to_device(inputs.uniform_lwe(p, 7711, 9))
    ref = ctx.bootstrap("ntt", cts)
    out = torch.full_like(ref, MARK)
    torch.cuda.synchronize()
    ctx.latency_abort()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        ctx.bootstrap("int8", cts, out)
    ctx.bootstrap("int8", cts, out)
    torch.cuda.synchronize()
    assert bool((out == MARK).all())
    with pytest.raises(cggi.CggiError):
        ctx.check()
    for _ in range(3):
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(out, ref)
        out.fill_(MARK)
        assert torch.equal(ctx.bootstrap("int8", cts), ref)
    del graph
    ctx.check()
    ctx.close()
