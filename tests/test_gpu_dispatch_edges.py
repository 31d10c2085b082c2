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


@pytest.mark.parametrize("C,heads,dtype", [(192, 8, "bf16"), (128, 8, "bf16"), (64, 4, "bf16"), (64, 4, "f32")])
@pytest.mark.parametrize("n_multi,n_single", [(0, 24577), (1, 24623), (8193, 9000), (12289, 0), (20, 24576 + 47)])
def test_pool_regions_of_one_voxel_apart(C, heads, dtype, n_multi, n_single):
    """Frames above and around the size from which regions of one voxel are taken apart: only such regions, none,
    a remainder of either kind; with the scratch the size call names and with the plain layout's, the same result.
    A call below the size (24,576 voxels) asks for the plain layout only."""
    grid, pool = (128, 128, 8), (1, 1, 4)
    rng = np.random.Generator(np.random.Philox(21))
    reg = rng.permutation(128 * 128 * 2)[:n_multi + n_single]
    rows = []
    for k, r in enumerate(reg):
        z = rng.permutation(4)[:1 if k >= n_multi else 2 + k % 3]
        rows += [(0, r // 256, r // 2 % 128, 4 * (r % 2) + int(v)) for v in z]
    coords = np.array(rows, np.int32)[rng.permutation(len(rows))]
    n = len(coords)
    x = synth.make_features(22, n, C, dtype)
    w = synth.make_pool_weights(23, C, heads, dtype)
    print(f"[case] pool apart C={C} {dtype} regions {n_multi} + {n_single}, {n} voxels", flush=True)
    ref_c, ref = orc.attn_pool(w, coords, x, grid, pool, 1)
    pw, plain = dsvt.PoolWeights(w, grid, pool, 1, 1), dsvt.PoolWeights(w, grid, pool, 1, 0)
    sizes = [dsvt.dsvt_attn_pool_workspace_size(p, n) for p in (pw, plain)]
    assert sizes[0] >= sizes[1] and (n > 24576 or sizes[0] == sizes[1])
    cd, xd, outs = dev_coords(coords), dev_feats(x, dtype), []
    for size in sizes:
        oc, out, n_out, status = dsvt.dsvt_attn_pool(pw, cd, xd, ws=torch.full((size,), 0x5A, dtype=torch.uint8, device="cuda"))
        torch.cuda.synchronize()
        assert int(status.item()) == 0 and int(n_out.item()) == len(ref_c) == n_multi + n_single
        assert np.array_equal(oc[:len(ref_c)].cpu().numpy(), ref_c)
        assert rel_err(out[:len(ref_c)], ref) < TOL[dtype]
        assert torch.all(out[len(ref_c):] == 0)
        outs.append(out)
    assert rel_err(outs[0], outs[1].double().cpu().numpy()) < TOL[dtype]


@pytest.mark.parametrize("C,heads,hidden,dtype", [(192, 8, 384, "bf16"), (64, 4, 128, "f32")])
@pytest.mark.parametrize("rows", [1, 16, 17, 33, 49, 65, 81, 96])
def test_layer_tiles_of_one_to_six_row_tiles(C, heads, hidden, dtype, rows):
    """One tile with every number of 16-row tiles: the LayerNorm phases split them unevenly over two halves, and in a
    tile of one the second half has nothing."""
    grid, win, tau = (12, 12, 1), (12, 12, 1), 96
    cell = np.random.Generator(np.random.Philox(31)).permutation(144)[:rows]
    coords = np.stack([0 * cell, cell // 12, cell % 12, 0 * cell], 1).astype(np.int32)
    x = synth.make_features(32, rows, C, dtype)
    ws = [synth.make_layer_weights(33 + a, C, heads, hidden, win, dtype) for a in (0, 1)]
    print(f"[case] one tile of {rows} rows C={C} {dtype}", flush=True)
    oms = [orc.partition(coords, grid, win, (0, 0, 0), tau, a) for a in (0, 1)]
    cd = dev_coords(coords)
    gms = [gpu_maps(cd, grid, win, (0, 0, 0), tau, 1, a) for a in (0, 1)]
    out = dsvt.dsvt_block([dsvt.LayerWeights(w) for w in ws], gms, cd, dev_feats(x, dtype))
    torch.cuda.synchronize()
    assert rel_err(out, orc.block(ws, oms, coords, x)) < TOL[dtype]
