"""The forms on their own kernels.  Where the transform kernel serves, the
tests of both forms, of latency mode and of the large set run on that one
kernel; here their bodies run on contexts made without it, which is also what a
context falls back to when the transforms find no room in memory.  The two
sides of every comparison between the forms are then different kernels: the
modular transform, and the int8 kernels under the built-in plan."""
import functools

import pytest

import test_gpu_golden as golden
import test_gpu_large as large
import test_gpu_latency as latency
import test_gpu_level as level
import test_gpu_parity as parity
import test_gpu_pbs as pbs
import test_zz_no_alloc as noalloc
from conftest import real_keys
from paper_2306_11006_amd import cggi, inputs, params

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True)
def own(monkeypatch):
    monkeypatch.setattr(cggi, "Context",
                        functools.partial(cggi.Context, transform=False))


def uniform(p, seed):
    bsk, ksk = inputs.uniform_keys(p, seed)
    ctx = cggi.Context(p, cggi.to_device(bsk), cggi.to_device(ksk))
    assert ctx.transform_width("ntt") == ctx.transform_width("int8") == 0
    return p, bsk, ksk, ctx


def real(p, seed):
    keys = real_keys(p, seed)
    ctx = cggi.Context(p, cggi.to_device(keys["bsk"]),
                       cggi.to_device(keys["ksk"]))
    assert ctx.transform_width("ntt") == ctx.transform_width("int8") == 0
    return p, keys, ctx


@pytest.mark.parametrize("p,batches", latency.CASES,
                         ids=[c[0].name for c in latency.CASES])
def test_latency_mode_bit_exact(O, p, batches):
    latency.test_latency_mode_bit_exact(O, p, batches)


@pytest.mark.parametrize("body", [
    latency.test_latency_mode_limits,
    latency.test_latency_mode_repeated_launches_and_graph,
    latency.test_latency_mode_abort_and_recovery,
    latency.test_latency_mode_contexts_of_different_sizes,
    noalloc.test_noalloc_matches_eval_level_two_calls,
    noalloc.test_noalloc_graph_replays], ids=lambda f: f.__name__)
def test_body(body):
    body()


@pytest.mark.parametrize("body", [
    golden.test_level_1024_nand_keygen_every_row,
    golden.test_adder_multiplier_default_every_wire,
    golden.test_mixed_level_16384_every_row,
    level.test_level_default_sizes_mixed_gates,
    large.test_large_real_key_gates], ids=lambda f: f.__name__)
def test_body_against_the_oracle(O, body):
    body(O)


@pytest.mark.parametrize("pset", ["toy", "default"])
def test_lookup_tables(O, pset):
    pbs.test_lut_bootstrap_bit_exact(O, pset, 4)


def test_toy_test_vector_and_levels(O):
    toy = real(params.TOY, 1)
    parity.test_toy_custom_test_vector(O, toy)
    level.test_level_every_gate_bit_exact_toy(O, toy)
    level.test_level_invalid_gates_are_skipped(O, toy)
    level.test_level_graph_replay_matches_eager(O, toy)
    toy[2].close()


def test_default_widths(O):
    default = uniform(params.DEFAULT, 2024)
    parity.test_default_ragged_small_batch(O, default)
    parity.test_default_full_batch_forms_agree_and_match_oracle(O, default)
    for B in (200, 400, 700):
        parity.test_default_batch_widths_pick_tiles(O, default, B)
    default[3].close()


def test_large_set(O):
    big = uniform(params.LARGE, 2048)
    large.test_large_bootstrap_bit_exact(O, big)
    large.test_large_forms_agree_batch(big)
    large.test_large_random_dag(O, big)
    big[3].close()
