"""Timed cases of the batched gate bootstrapping library.

Every case is one pass through the public entry points
(paper_2306_11006_amd.cggi.Context, circuit.LevelledCircuit) at one of the
repository's parameter sets.  Kinds of pass ("op"):

* level     -- one cggi_eval_level of independent gates;
* bootstrap -- one batch of (programmable) bootstraps, big ciphertexts out;
* lut       -- a programmable bootstrap with a lookup-table test polynomial,
               then the key switch: the table lookup of a user's program;
* keyswitch -- one batch of key switches;
* circuit   -- a levelled circuit run level by level;
* graph     -- the same circuit as one captured HIP graph, replayed.

Keys and ciphertexts are uniform words drawn on the GPU from the seed: under
the LWE assumption real ones cannot be told from these, and no kernel's work
depends on their values.
"""
import math

import numpy as np
import torch

from paper_2306_11006_amd import arith, cggi, inputs, params, pbs
from paper_2306_11006_amd.circuit import LevelledCircuit

# opcode numbers of the C ABI
NAND, AND, OR, XOR, MUX = 0, 1, 2, 3, 4
MU = 1 << 29
MIXED_OPS = (NAND, AND, OR, XOR, MUX)


def listed():
    return [
        # the toy workload: four NANDs, one per input pair; launches and
        # per-step latency are all there is
        dict(name="toy_4_nand", op="level", set="toy", form="int8", width=4,
             mix=False),
        # a single encrypted gate: the narrowest level of any circuit
        dict(name="one_nand", op="level", set="default", form="int8",
             width=1, mix=False),
        # a 32-bit prefix adder called level by level: seven narrow levels
        dict(name="add32_prefix", op="circuit", set="default", form="int8",
             circuit="adder", style="prefix", bits=32),
        # a table lookup on a ragged batch of small messages
        dict(name="lut_100", op="lut", set="default", form="int8", width=100,
             msg=8),
        # the benchmark's level, in both forms
        dict(name="nand_1024", op="level", set="default", form="int8",
             width=1024, mix=False),
        dict(name="nand_1024_ntt", op="level", set="default", form="ntt",
             width=1024, mix=False),
        # the wide mixed level (19.7k bootstraps)
        dict(name="mixed_16384", op="level", set="default", form="int8",
             width=16384, mix=True),
        # the uneven circuit as programs run it for throughput: captured
        # once, replayed (88 levels of 1 to 273 gates)
        dict(name="uneven_16bit", op="graph", set="default", form="int8",
             circuit="uneven", style="ripple", bits=16),
        # the large set in the form its autotuner picks: a narrow level and
        # a wide one of the random DAG
        dict(name="large_mixed_37", op="level", set="large", form="ntt",
             width=37, mix=True),
        dict(name="large_mixed_2000", op="level", set="large", form="ntt",
             width=2000, mix=True),
        # bootstraps of the large set in the other form, a ragged batch
        dict(name="large_300", op="bootstrap", set="large", form="int8",
             width=300),
        # key switches alone
        dict(name="keyswitch_1024", op="keyswitch", set="default",
             form="int8", width=1024),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


# widest batch drawn per parameter set (no drawn case costs more than the
# widest listed level)
_WIDEST = {"toy": 16384, "default": 12000, "large": 2000}


def draw(rng):
    s = rng.choice(["toy", "default", "default", "default", "large"])
    op = rng.choice(["level", "level", "bootstrap", "lut", "keyswitch",
                     "circuit", "graph"])
    form = rng.choice(["int8", "ntt"])
    case = dict(op=op, set=s, form=form)
    if op in ("circuit", "graph"):
        kind = rng.choice(["adder", "adder", "multiplier"])
        case["circuit"] = kind
        case["style"] = rng.choice(["ripple", "prefix"] if kind == "adder"
                                   else ["array", "tree"])
        if s == "large" or form == "ntt":
            # the slowest combinations stay below the widest listed level
            case["style"] = "prefix" if kind == "adder" else "tree"
            case["bits"] = rng.randint(3, 6 if kind == "multiplier" else 14)
        else:
            case["bits"] = rng.randint(3, 9 if kind == "multiplier" else 32)
        return case
    hi = _WIDEST[s]
    if s == "large" and form == "int8":
        hi = 1000
    elif form == "ntt" and s == "default":
        hi = 8000
    case["width"] = _log_int(rng, 1, hi)
    if op == "level":
        case["mix"] = rng.random() < 0.7
    elif op == "lut":
        case["msg"] = rng.choice([2, 4, 8])
    elif op == "keyswitch":
        case["width"] = _log_int(rng, 1, 16384)
    return case


# ---- inputs ----------------------------------------------------------------

def _words(gen, *shape):
    """Uniform 32-bit words as an int32 tensor on the GPU."""
    return torch.randint(-(1 << 31), 1 << 31, shape, dtype=torch.int32,
                         device="cuda", generator=gen)


def _keys(p, seed):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(2 * seed + 1)
    return _words(gen, *p.bsk_shape), _words(gen, *p.ksk_shape)


def _input_words(seed, *shape):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(2 * seed + 2)
    return _words(gen, *shape)


def _level_gates(case, seed):
    """Gates of a level: gate g reads wires 3g .. 3g + 2, writes 3W + g."""
    w = case["width"]
    idx = np.arange(w, dtype=np.int32)
    if case["mix"]:
        ops = np.random.default_rng(seed).choice(MIXED_OPS, size=w)
    else:
        ops = np.full(w, NAND)
    return np.stack([ops, 3 * idx, 3 * idx + 1, 3 * idx + 2, 3 * w + idx],
                    axis=1).astype(np.int32)


def _netlist(case):
    """(gates, number of wires, input wires) of a circuit case."""
    if case["circuit"] == "uneven":
        nl, io = inputs.adder_multiplier_circuit(case["bits"])
    elif case["circuit"] == "adder":
        nl, io = arith.adder(case["bits"], case["style"])
    else:
        nl, io = arith.multiplier(case["bits"], case["style"])
    return nl.array(), nl.n_wires, list(nl.input_wires)


def _lut(msg, seed):
    return [int(v) for v in np.random.default_rng(seed).integers(0, msg, msg)]


def _circuit_wires(p, n_wires, ins, seed):
    wires = torch.zeros((n_wires, p.n + 1), dtype=torch.int32, device="cuda")
    wires[torch.tensor(ins, device="cuda")] = \
        _input_words(seed, len(ins), p.n + 1)
    return wires


class _State:
    pass


def prepare(case, seed):
    p = params.ALL[case["set"]]
    bsk, ksk = _keys(p, seed)
    st = _State()
    st.case = case
    st.ctx = cggi.Context(p, bsk, ksk, forms=(case["form"],))
    op = case["op"]
    if op == "level":
        w = case["width"]
        st.gates = cggi.to_device(_level_gates(case, seed))
        st.wires = torch.zeros((4 * w, p.n + 1), dtype=torch.int32,
                               device="cuda")
        st.wires[:3 * w] = _input_words(seed, 3 * w, p.n + 1)
        st.ctx.reserve(w)
    elif op in ("circuit", "graph"):
        gates, n_wires, ins = _netlist(case)
        st.circ = LevelledCircuit(gates, n_wires)
        st.wires = _circuit_wires(p, n_wires, ins, seed)
        st.ctx.reserve(max(st.circ.widths))
        if op == "graph":
            st.graph = st.circ.capture(st.ctx, case["form"], st.wires)
    elif op == "keyswitch":
        st.big = _input_words(seed, case["width"], p.N + 1)
        st.out = torch.empty((case["width"], p.n + 1), dtype=torch.int32,
                             device="cuda")
    else:
        st.cts = _input_words(seed, case["width"], p.n + 1)
        st.big = torch.empty((case["width"], p.N + 1), dtype=torch.int32,
                             device="cuda")
        if op == "lut":
            st.testv = cggi.to_device(pbs.lut_test_vector(
                _lut(case["msg"], seed), case["msg"], p.N))
            st.out = torch.empty((case["width"], p.n + 1), dtype=torch.int32,
                                 device="cuda")
    return st


def run(st):
    case, ctx = st.case, st.ctx
    op, form = case["op"], case["form"]
    if op == "level":
        return ctx.eval_level(form, st.gates, st.wires)
    if op == "circuit":
        return st.circ.run(ctx, form, st.wires)
    if op == "graph":
        st.graph.replay()
        return st.wires
    if op == "keyswitch":
        return ctx.keyswitch(st.big, st.out)
    if op == "lut":
        ctx.bootstrap(form, st.cts, st.big, testv=st.testv)
        ctx.keyswitch(st.big, st.out)
        return [st.big, st.out]
    return ctx.bootstrap(form, st.cts, st.big)


# ---- work ------------------------------------------------------------------

def _counts(case):
    """(bootstraps, key switches, ciphertext words in and out) of a pass."""
    p = params.ALL[case["set"]]
    n1, N1 = p.n + 1, p.N + 1
    op = case["op"]
    if op in ("circuit", "graph"):
        gates, _, ins = _netlist(case)
        bs = LevelledCircuit._bootstraps(gates)
        ks = int(np.isin(gates[:, 0], (0, 1, 2, 3, 4, 9, 10)).sum())
        return bs, ks, (len(ins) + len(gates)) * n1
    w = case["width"]
    if op == "level":
        # mixed gates: a fifth are MUX (two bootstraps, three inputs)
        bs = round(w * 1.2) if case["mix"] else w
        return bs, w, (round(w * 2.2) if case["mix"] else 2 * w) * n1 + w * n1
    if op == "keyswitch":
        return 0, w, w * (N1 + n1)
    if op == "lut":
        return w, w, w * (n1 + N1 + N1 + n1) + p.N
    return w, 0, w * (n1 + N1)


def work(case):
    """The key material read once and the ciphertexts in and out; the
    operations of a blind rotation whose products are done by transforms of
    half the ring degree (2l forward and two back per step), and the sums
    of the key switch's rows."""
    p = params.ALL[case["set"]]
    bs, ks, words = _counts(case)
    nbytes = 4 * words
    flops = 0
    if bs:
        nbytes += 4 * p.n * 2 * p.l * 2 * p.N
        h = p.N // 2
        per_step = ((2 * p.l + 2) * 5 * h * int(math.log2(h)) +
                    2 * p.l * 2 * 8 * h)
        flops += bs * p.n * per_step
    if ks:
        rows = p.N * p.ks_t * p.ks_base
        # a few ciphertexts read only the rows their digits name
        nbytes += 4 * (p.n + 1) * min(rows, ks * p.N * p.ks_t)
        flops += ks * p.N * p.ks_t * (p.n + 1)
    return {"bytes": int(nbytes), "flops": int(flops)}


# ---- the same results in plain torch, 64-bit arithmetic --------------------

M32 = 0xFFFFFFFF


def _wrap(x):
    """int64 -> int32 with the same low 32 bits."""
    x = x & M32
    return torch.where(x >= 1 << 31, x - (1 << 32), x).to(torch.int32)


def _u(t):
    """int32 words -> int64 in [0, 2^32)."""
    return t.to(torch.int64) & M32


def _exact_bootstrap(p, bsk, cts, testv):
    """Fig. 1's loop on int64 words; each step's products as one float64
    matrix product per 16-bit half of the key, exact (every sum is an
    integer below 2^53)."""
    dev = cts.device
    n, N, l, beta = p.n, p.N, p.l, p.bg_bit
    B = cts.shape[0]
    logn = (2 * N).bit_length() - 1
    ms = ((_u(cts) + (1 << (31 - logn))) & M32) >> (32 - logn)
    idx = torch.arange(N, device=dev)

    def rotate(x, e):
        """X^e x for polynomials x [B, c, N] and exponents e [B]."""
        t = (idx[None, :] - e[:, None]) % (2 * N)
        v = torch.gather(x, 2, (t % N)[:, None, :].expand(-1, x.shape[1], -1))
        return torch.where((t >= N)[:, None, :], -v, v)

    acc = torch.zeros((B, 2, N), dtype=torch.int64, device=dev)
    acc[:, 1] = testv
    acc = rotate(acc, (2 * N - ms[:, n]) % (2 * N)) & M32
    off = 1 << (31 - beta * l) if beta * l < 32 else 0
    for q in range(1, l + 1):
        off += (1 << (beta - 1)) << (32 - q * beta)
    # Toeplitz row m, column j holds a[j - m], negated when it wraps
    d = idx[None, :] - idx[:, None]
    pos, sign = d % N, torch.where(d < 0, -1.0, 1.0).to(torch.float64)
    for i in range(n):
        w = (rotate(acc, ms[:, i]) - acc + off) & M32
        dig = torch.stack([((w >> (32 - q * beta)) & ((1 << beta) - 1)) -
                           (1 << (beta - 1)) for q in range(1, l + 1)], 2)
        dig = dig.reshape(B, 2 * l * N).to(torch.float64)
        a = _u(bsk[i])                                   # [2l, 2, N]
        for half in (0, 1):
            h = ((a >> (16 * half)) & 0xFFFF).to(torch.float64)
            m = (h[:, :, pos] * sign).permute(0, 2, 1, 3)
            r = dig @ m.reshape(2 * l * N, 2 * N)
            acc += r.to(torch.int64).reshape(B, 2, N) << (16 * half)
        acc &= M32
    out = torch.empty((B, N + 1), dtype=torch.int64, device=dev)
    out[:, 0] = acc[:, 0, 0]
    out[:, 1:N] = -acc[:, 0, 1:].flip(1)
    out[:, N] = acc[:, 1, 0]
    return out & M32


def _exact_keyswitch(p, ksk, big):
    g, t = p.ks_base_bit, p.ks_t
    rows = _u(ksk).reshape(p.N * t * p.ks_base, p.n + 1)
    off = 1 << (31 - t * g) if t * g < 32 else 0
    a = (big[:, :p.N] + off) & M32
    out = torch.zeros((big.shape[0], p.n + 1), dtype=torch.int64,
                      device=big.device)
    out[:, p.n] = big[:, p.N]
    base = torch.arange(p.N, device=big.device) * t
    for q in range(t):
        d = (a >> (32 - (q + 1) * g)) & (p.ks_base - 1)
        pick = (base + q) * p.ks_base + d                # [B, N]
        for b in range(big.shape[0]):
            out[b] -= rows[pick[b]].sum(0)
    return out & M32


def _exact_level(p, bsk, ksk, gates, wires):
    """One level on int64 wires, in place; gates of the circuits' opcodes."""
    def trivial(c):
        v = torch.zeros(p.n + 1, dtype=torch.int64, device=wires.device)
        v[p.n] = c
        return v

    pre, owner = [], []
    consts = {7: -MU, 8: MU}
    for k, (op, a, b, c, o) in enumerate(gates.tolist()):
        x, y, z = wires[a], wires[b], wires[c]
        if op in consts:
            wires[o] = trivial(consts[op]) & M32
            continue
        if op == NAND:
            ins = [trivial(MU) - x - y]
        elif op == AND:
            ins = [trivial(-MU) + x + y]
        elif op == OR:
            ins = [trivial(MU) + x + y]
        elif op == XOR:
            ins = [trivial(2 * MU) + 2 * (x + y)]
        elif op == MUX:
            ins = [trivial(-MU) + x + y, trivial(-MU) - x + z]
        else:
            raise ValueError(op)
        owner.append((o, len(pre), len(ins)))
        pre += ins
    if not pre:
        return
    testv = torch.full((p.N,), MU, dtype=torch.int64, device=wires.device)
    big = _exact_bootstrap(p, bsk, _wrap(torch.stack(pre)), testv)
    rows = []
    for o, s, k in owner:
        v = big[s]
        if k == 2:
            v = v + big[s + 1]
            v[p.N] += MU
        rows.append(v & M32)
    res = _exact_keyswitch(p, ksk, torch.stack(rows))
    wires[torch.tensor([o for o, _, _ in owner], device=wires.device)] = res


def exact(case, seed):
    p = params.ALL[case["set"]]
    op = case["op"]
    bs, ks, _ = _counts(case)
    steps = p.n
    if op in ("circuit", "graph"):
        gates, n_wires, ins = _netlist(case)
        circ = LevelledCircuit(gates, n_wires)
        steps *= circ.n_levels
    # seconds: matrix products, Toeplitz matrices of each step, key switch
    size = 2.0 * p.l * p.N * 2 * p.N
    cost = (4 * size * p.n * bs / 2e13 + 40 * size * steps / 2e12 +
            1e-4 * p.ks_t * ks)
    if cost > 12.0:
        return None
    bsk, ksk = _keys(p, seed)
    if op in ("circuit", "graph"):
        wires = _u(_circuit_wires(p, n_wires, ins, seed))
        for lv in circ.levels:
            _exact_level(p, bsk, ksk, lv, wires)
        return _wrap(wires)
    w = case["width"]
    if op == "level":
        wires = torch.zeros((4 * w, p.n + 1), dtype=torch.int64,
                            device="cuda")
        wires[:3 * w] = _u(_input_words(seed, 3 * w, p.n + 1))
        _exact_level(p, bsk, ksk, _level_gates(case, seed), wires)
        return _wrap(wires)
    if op == "keyswitch":
        big = _u(_input_words(seed, w, p.N + 1))
        return _wrap(_exact_keyswitch(p, ksk, big))
    cts = _input_words(seed, w, p.n + 1)
    if op == "lut":
        testv = torch.from_numpy(
            _lut_words(_lut(case["msg"], seed), case["msg"], p.N)).to("cuda")
    else:
        testv = torch.full((p.N,), MU, dtype=torch.int64, device="cuda")
    big = _exact_bootstrap(p, bsk, cts, testv)
    if op == "lut":
        return [_wrap(big), _wrap(_exact_keyswitch(p, ksk, big))]
    return _wrap(big)


def _lut_words(table, msg, N):
    """Test polynomial of a table over Z_msg with one padding bit: boxes of
    N / msg coefficients centred on each message, the lower half box of 0
    reached through the negacyclic wrap."""
    box, step = N // msg, (1 << 32) // (2 * msg)
    m = (np.arange(N) + box // 2) // box
    v = np.where(m < msg, np.take(table, np.minimum(m, msg - 1)) * step,
                 -table[0] * step)
    return v.astype(np.int64) & M32
