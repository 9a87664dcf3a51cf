"""The transform kernel where its build, its row layout or its dispatch
changes, beyond the sets of test_gpu_fft.py.  Tolerance 0 against the oracle:
the results are integers."""
import pytest

import test_gpu_fft as F

pytestmark = pytest.mark.gpu

# run-time digit counts: two rows a turn at the rings that lacked one, and the
# workgroup that takes all 160 KB of LDS
RUNTIME = [F.case(33, 512, 6, 4), F.case(9, 512, 9, 1), F.case(6, 2048, 7, 4),
           F.case(67, 256, 3, 8), F.case(5, 1024, 5, 6)]


@pytest.mark.parametrize("p", RUNTIME, ids=[p.name for p in RUNTIME])
def test_run_time_digit_counts(O, p):
    assert F.bound(p) <= 0.25
    F.check(O, p, ("ntt",), 9500 + RUNTIME.index(p), 5, False)
    F.check(O, p, ("ntt",), 9520 + RUNTIME.index(p), 3, True)


# (set, int8 bootstraps per CU up to which the transform kernel serves; None:
# every width)
WIDTHS = [(F.case(3, 256, 7, 3), 6), (F.case(3, 256, 7, 1), 2),
          (F.case(2, 512, 7, 2), 6), (F.case(2, 512, 7, 1), 1),
          (F.case(3, 512, 6, 4), None), (F.case(3, 256, 8, 2), None)]


@pytest.mark.parametrize("p,per_cu", WIDTHS, ids=[c[0].name for c in WIDTHS])
def test_int8_width_of_the_transform_kernel(O, p, per_cu):
    """The int8 form's batches on both sides of the widest one the transform
    kernel takes, with a count known on the host and one read on the device."""
    import numpy as np
    import torch
    from paper_2306_11006_amd import cggi, inputs
    seed = 9600 + p.N + p.l
    bsk, ksk = inputs.uniform_keys(p, seed)
    ctx = cggi.Context(p, cggi.to_device(bsk), cggi.to_device(ksk))
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    width = ctx.transform_width("int8")
    assert width == (cggi.INT32_MAX if per_cu is None else per_cu * cus)
    assert ctx.transform_width("ntt") == cggi.INT32_MAX
    top = width if per_cu else 2 * cus
    cts = inputs.uniform_lwe(p, seed + 1, top + 1)
    with F.cf.ThreadPoolExecutor(F.THREADS) as ex:
        want = np.stack(list(ex.map(lambda x: O.bootstrap(p, bsk, x), cts)))
    d_cts = cggi.to_device(cts)
    for B in (top, top + 1):
        print(f"width {p.name} B={B}", file=F.sys.stderr, flush=True)
        out = ctx.bootstrap("int8", d_cts[:B])
        assert np.array_equal(cggi.to_host(out), want[:B]), B
    # levels of NAND gates padded with copies: 2G bounds the count from above
    for B in (top, top + 1):
        W = 2 * (top + 8)
        wires = inputs.uniform_lwe(p, seed + 2, W)
        g = np.zeros((B + 7, 5), dtype=np.int32)
        g[B:, 0] = cggi.OPCODES["COPY"]
        g[:, 1] = np.arange(B + 7) % (top // 2)
        g[:, 2] = top // 2
        g[:, 4] = W // 2 + np.arange(B + 7)
        got = {}
        for form in ("int8", "ntt"):
            print(f"level {p.name} B={B} form={form}", file=F.sys.stderr,
                  flush=True)
            w = cggi.to_device(wires)
            ctx.eval_level(form, cggi.to_device(g), w)
            got[form] = cggi.to_host(w)
        assert np.array_equal(got["int8"], got["ntt"]), B
        for k in (0, B - 1):
            pre = O.gate_preop(p.n, "NAND", wires[g[k, 1]], wires[g[k, 2]])
            out = O.keyswitch(p, ksk, O.bootstrap(p, bsk, pre))
            assert np.array_equal(got["int8"][g[k, 4]], out), (B, k)
    ctx.check()
    ctx.close()


@pytest.mark.parametrize("B", [257, 600])
def test_two_bootstraps_per_workgroup_at_two_levels(O, B):
    F.check(O, F.case(4, 1024, 10, 2), ("ntt",), 9700 + B, B, False)


@pytest.mark.parametrize("p", F.INSIDE + F.PAST,
                         ids=[p.name for p in F.INSIDE + F.PAST])
def test_which_kernel_serves(p):
    from paper_2306_11006_amd import cggi, inputs
    bsk, ksk = inputs.uniform_keys(p, 9750)
    ctx = cggi.Context(p, cggi.to_device(bsk), cggi.to_device(ksk),
                       forms=("ntt",))
    assert ctx.transform_width("ntt") == (cggi.INT32_MAX if p in F.INSIDE
                                          else 0)
    ctx.close()


@pytest.mark.parametrize("l", [2, 3])
def test_device_counts_around_the_pairs(O, l):
    """Levels whose bootstrap count, known on the device only, fills rounds of
    two bootstraps per workgroup and leaves a rest on either side of half a
    round (MUX gates: two bootstraps each)."""
    import numpy as np
    import torch
    from paper_2306_11006_amd import cggi, inputs
    p = F.case(4, 1024, 7, l)
    bsk, ksk = inputs.uniform_keys(p, 9760 + l)
    ctx = cggi.Context(p, cggi.to_device(bsk), cggi.to_device(ksk))
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    for count in (1, cus, cus + 1, 2 * cus, 2 * cus + 1, 3 * cus,
                  3 * cus + 1):
        mux = min(count // 2, 40)
        G = count - mux + 5                     # and five copies
        wires = inputs.uniform_lwe(p, 9770 + count, 64 + G)
        g = inputs.rng(9780 + count).integers(0, 64, size=(G, 5))
        g[:, 0] = cggi.OPCODES["NAND"]
        g[:mux, 0] = cggi.OPCODES["MUX"]
        g[-5:, 0] = cggi.OPCODES["COPY"]
        g[:, 4] = 64 + np.arange(G)
        g = g.astype(np.int32)
        with F.cf.ThreadPoolExecutor(F.THREADS) as ex:
            want = np.stack(list(ex.map(
                lambda t: O.gate(p, int(t[0]), bsk, ksk, wires[t[1]],
                                 wires[t[2]], wires[t[3]]), g)))
        for form in ("int8", "ntt"):
            print(f"level {p.name} count={count} form={form}",
                  file=F.sys.stderr, flush=True)
            w = cggi.to_device(wires)
            ctx.eval_level(form, cggi.to_device(g), w)
            got = cggi.to_host(w)
            assert np.array_equal(got[64:], want), (count, form)
            assert np.array_equal(got[:64], wires[:64])
    ctx.close()
