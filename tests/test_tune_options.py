"""The tuner times and reports launches, not option values that launch the same: at most 4 workgroups of the
persistent form are resident per compute unit, and more are not launched."""
import ctypes

import numpy as np
import pytest
import torch  # before the library: both use its HIP runtime

from paper_2606_05581_amd import workloads as W


def test_default_space_names_each_launch_once():
    from paper_2606_05581_amd import msk

    sp = msk.TuneSpace()
    msk.lib().msk_tune_space_default(ctypes.byref(sp))
    launched = [min(4, sp.blocks_per_cu[i]) for i in range(sp.n_bpc)]
    assert launched and len(set(launched)) == len(launched)


@pytest.mark.gpu
def test_tuner_times_each_launch_once_and_reports_it(tmp_path):
    from paper_2606_05581_amd import msk

    ctx = msk.Context(0)
    V, F = W.icosphere_recursive(2)
    case = W._point_case(V, F, 50, np.random.default_rng(0))
    mesh = ctx.build_bvh(case.V, case.F)
    args = ([mesh], [ctx.rows(mesh, case.rows)], [ctx.basis(case.basis, case.V.shape[0])], [case.eps], [case.h])
    space = dict(trial_rows=50, trial_walks=16, repeats=1, leaf=[4], chunk=[64], regen_min=[16])
    one = ctx.autotune(*args, **space, blocks_per_cu=[4])
    path = str(tmp_path / "cache.jsonl")
    more = ctx.autotune(*args, **space, blocks_per_cu=[4, 8, 16], cache_path=path)
    assert more["trials"] == one["trials"] and more["blocks_per_cu"] == one["blocks_per_cu"] == 4
    two = ctx.autotune(*args, **space, blocks_per_cu=[2, 4])
    assert two["trials"] == one["trials"] + 1 and two["blocks_per_cu"] in (2, 4)
    # a stored setting of 8 workgroups is read as the 4 that it launches
    text = open(path).read()
    assert '"blocks_per_cu": 4' in text
    open(path, "w").write(text.replace('"blocks_per_cu": 4', '"blocks_per_cu": 8'))
    again = ctx.autotune(*args, **space, cache_path=path)
    assert again["from_cache"] and again["blocks_per_cu"] == 4
    ctx.close()
