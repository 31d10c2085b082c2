"""Kernel variants and dispatch rules at the sizes where they can go wrong, against the CPU oracle."""
import numpy as np
import pytest
import torch

import synth
from oracle import dsvt_oracle as orc

pytestmark = pytest.mark.gpu
dsvt = pytest.importorskip("paper_2301_06051_amd")
from gpu_util import TOL, dev_coords, dev_feats, gpu_maps, rel_err  # noqa: E402


@pytest.mark.parametrize("C,heads,hidden,dtype", [(192, 8, 384, "bf16"), (128, 8, 256, "bf16"), (64, 4, 128, "f32")])
@pytest.mark.parametrize("dup_mode", [0, 1])
def test_large_sets_heads_per_item(C, heads, hidden, dtype, dup_mode):
    """Sets of four to six key tiles (full windows of 64, 65, 80, 81 and 96 voxels): items of one or two heads."""
    grid, win, tau = (60, 12, 1), (12, 12, 1), 96
    rng = np.random.Generator(np.random.Philox(11))
    rows = []
    for k, cnt in enumerate((64, 65, 80, 81, 96)):
        cell = rng.permutation(144)[:cnt]
        rows.append(np.stack([0 * cell, 12 * k + cell // 12, cell % 12, 0 * cell], 1))
    coords = np.concatenate(rows).astype(np.int32)
    x = synth.make_features(12, len(coords), C, dtype)
    w = synth.make_layer_weights(13, C, heads, hidden, win, dtype)
    print(f"[case] large sets C={C} {dtype} dup={dup_mode}", flush=True)
    om = orc.partition(coords, grid, win, (0, 0, 0), tau, 0)
    cd = dev_coords(coords)
    y = dsvt.dsvt_set_attention(dsvt.LayerWeights(w, dup_mode), gpu_maps(cd, grid, win, (0, 0, 0), tau, 1, 0), cd, dev_feats(x, dtype))
    torch.cuda.synchronize()
    assert rel_err(y, orc.set_attention(w, om, coords, x, dup_mode)) < TOL[dtype]
