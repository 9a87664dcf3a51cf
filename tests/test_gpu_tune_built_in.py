"""The tuner times the built-in choice where the transform kernel serves: it is
faster than every int8 kernel at the toy set, so the tuned table keeps it, with
both forms in the context and with the int8 form alone."""
import pytest

from paper_2306_11006_amd import cggi, inputs, params, tune

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("forms", [("ntt", "int8"), ("int8",)],
                         ids=["both", "int8"])
def test_table_keeps_the_transform_kernel(forms):
    p = params.TOY
    bsk, ksk = inputs.uniform_keys(p, 8600)
    ctx = cggi.Context(p, cggi.to_device(bsk), cggi.to_device(ksk),
                       forms=forms)
    built_in = ctx.int8_plan_get()
    ctx.int8_plan([("tiles4", 1 << 24)])
    table = tune.autotune(ctx, p, widths=[1, 100, 1024], reps=2)
    assert ctx.transform_width("int8") == cggi.INT32_MAX
    assert table["plan"] == built_in
    for w in ("1", "100", "1024"):
        assert table["forms"][w]["int8"] == table["served"][w]
        assert table["served"][w] <= min(table["times"][w].values())
    tune.apply(ctx, table)
    assert ctx.transform_width("int8") == cggi.INT32_MAX
    assert ctx.int8_plan_get() == built_in
    ctx.close()
