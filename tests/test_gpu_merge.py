"""GPU merge of many key-range splits against the oracle: items of more than 16 splits in few rows take one row
per workgroup, with runs of neighbouring splits summed by groups of threads; split counts that leave the last
groups without a split, rows that do not fill an item, and items of few splits in the same launch or, when they
have many rows, in one of their own; items of many splits and many rows are walked by a thread a row."""
import pytest

import paper_2609_35263_amd as wp
import workloads as wl
from tests._harness import gpu_wave
from tests.test_gpu_parity import check_wave

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape,prefix,chunk,splits", [
    ((16, 4, 64, 64), [2171, 100], [5, 40], 17),       # one split more than the one-trip form takes
    ((16, 1, 64, 64), [17015], [9], 133),               # more splits than 16 groups x 8 loads
    ((16, 16, 128, 128), [2047, 300], [129, 1], 17),   # 8 groups, the last without a split
    ((64, 8, 128, 128), [11480], [40], 90),            # 8-wave items
    ((16, 1, 576, 512), [1085], [3], 17),              # latent: 4 groups
    ((128, 1, 576, 512), [8958, 50], [2, 1], 140),
    ((64, 8, 128, 128), [6000, 300], [2, 70], 47),     # 128 rows of 47 splits, 4,480 of 3: a launch each
    ((16, 1, 64, 64), [2560], [90], 21),               # 1,440 rows of 21 splits: a thread a row, splits by fours
    ((16, 1, 576, 512), [1100, 500], [40, 3], 18),     # the same, latent, with an item of few splits
])
def test_many_splits(shape, prefix, chunk, splits):
    import torch
    Hq, Hkv, dk, dv = shape
    spec = wl.custom_wave(Hq, Hkv, dk, dv, 64, prefix, chunk, kv_shared=dk == 576, seed=splits, name="merge")
    used = wp.plan_for(spec, max_splits=splits).info()["max_splits"]
    print(f"[merge] {shape} {prefix} {chunk} splits={used}", flush=True)
    assert used > 16
    g, _, t = check_wave(spec, seed=31 + splits, max_splits=splits)
    again = gpu_wave(spec, t, max_splits=splits)
    assert torch.equal(again["out"], g["out"]) and torch.equal(again["lse"], g["lse"])
