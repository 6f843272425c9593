"""The kernel-shape plan on the host: what a plan is set for, a launch takes it as it takes the
caller's opt->variant (seen here by the workspace it asks for)."""
import pytest

import paper_2511_11430_amd as vpm
from paper_2511_11430_amd import _lib


@pytest.fixture
def no_plans():
    from paper_2511_11430_amd import tune

    def clear():
        for b in (0, 1):
            assert _lib.load().vpm_set_plan(vpm.F32C, b, 0, 1 << 31, 0) == 0
    clear()
    yield
    clear()
    tune.apply_cache()


@pytest.mark.parametrize("off,variant", [([0, 20000], 1), ([0, 50000], 7), ([0, 100000], 4),
                                         ([0] + [9000 * k for k in range(1, 13)], 8)])
def test_a_plan_is_used_as_the_variant(off, variant, no_plans):
    batched = int(len(off) > 2)
    own = vpm.vpm_workspace_size(vpm.F32C, off)
    asked = vpm.vpm_workspace_size(vpm.F32C, off, variant=variant)
    gradient = vpm.vpm_workspace_size(vpm.F32C, off, gradient=True)
    f64 = vpm.vpm_workspace_size(vpm.F64, off)
    assert own != asked  # (the sizes tell the two apart)
    vpm.vpm_set_plan(batched, off[-1], off[-1], variant)
    assert vpm.vpm_get_plan(batched, off[-1]) == variant
    assert vpm.vpm_workspace_size(vpm.F32C, off) == asked
    # neither the gradient mode nor FP64 takes a plan
    assert vpm.vpm_workspace_size(vpm.F32C, off, gradient=True) == gradient
    assert vpm.vpm_workspace_size(vpm.F64, off) == f64
    vpm.vpm_set_plan(batched, off[-1], off[-1], 0)
    assert vpm.vpm_workspace_size(vpm.F32C, off) == own


def test_the_shipped_cache_holds_what_the_tuner_found():
    """Each plan is the fastest timing of its row, or 0 where the library's own spread ("0") is within 1 %."""
    import json
    from paper_2511_11430_amd import tune
    with open(tune.DEFAULT_CACHE) as f:
        plans = json.load(f)["plans"]
    for p in plans:
        ms = {int(k): t for k, t in p["ms"].items()}
        best = min((k for k in ms if k), key=lambda k: ms[k])
        assert p["variant"] == (best if ms[best] < tune.GAIN * ms[0] else 0)
        assert p["batched"] or p["n_lo"] >= tune.TUNED_FROM
