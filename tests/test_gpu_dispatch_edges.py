"""Kernel variants and dispatch rules at the sizes where they can go wrong, against the CPU oracle."""
import numpy as np
import pytest
import torch

import synth
from oracle import dsvt_oracle as orc

pytestmark = pytest.mark.gpu
dsvt = pytest.importorskip("paper_2301_06051_amd")
from gpu_util import TOL, dev_coords, dev_feats, gpu_maps, rel_err  # noqa: E402


@pytest.mark.parametrize("C,heads,hidden,dtype", [(192, 8, 384, "bf16"), (128, 8, 256, "bf16"), (64, 4, 128, "bf16"), (64, 4, 128, "f32")])
@pytest.mark.parametrize("dup_mode", [0, 1])
def test_large_sets_heads_per_item(C, heads, hidden, dtype, dup_mode):
    """Sets of four to six key tiles (full windows of 64, 65, 80, 81 and 96 voxels): items of one, two or four heads."""
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


@pytest.mark.parametrize("slope", [0.3, 9.0, 400.0])
@pytest.mark.parametrize("dup_mode", [0, 1])
def test_logits_that_rise_and_fall_over_a_large_set(slope, dup_mode):
    """C = 128 takes the keys of a large set 32 at a time with a running maximum: positional terms that rise along the set in half of the
    heads and fall in the others, by little, by about what exp2 takes from one 32 keys to the next, and by far more."""
    C, heads, grid, win, tau = 128, 8, (60, 12, 1), (12, 12, 1), 96
    rng = np.random.Generator(np.random.Philox(71))
    rows = []
    for k, cnt in enumerate((49, 64, 65, 81, 96)):
        cell = rng.permutation(144)[:cnt]
        rows.append(np.stack([0 * cell, 12 * k + cell // 12, cell % 12, 0 * cell], 1))
    coords = np.concatenate(rows).astype(np.int32)
    x = synth.make_features(72, len(coords), C, "bf16")
    w = synth.make_layer_weights(73, C, heads, 256, win, "bf16")
    dx = np.arange(23 * 23) // 23 - 11                       # query - key
    w["rel_bias"] = (slope * dx[None, :] * np.where(np.arange(heads) % 2 == 0, 1, -1)[:, None]).astype(np.float32)
    print(f"[case] rising and falling logits slope={slope} dup={dup_mode}", flush=True)
    om = orc.partition(coords, grid, win, (0, 0, 0), tau, 0)
    cd = dev_coords(coords)
    y = dsvt.dsvt_set_attention(dsvt.LayerWeights(w, dup_mode), gpu_maps(cd, grid, win, (0, 0, 0), tau, 1, 0), cd, dev_feats(x, "bf16"))
    torch.cuda.synchronize()
    assert rel_err(y, orc.set_attention(w, om, coords, x, dup_mode)) < TOL["bf16"]


@pytest.mark.parametrize("C,heads,hidden,dtype", [(192, 8, 384, "bf16"), (128, 8, 256, "bf16"), (64, 4, 128, "bf16"), (64, 4, 128, "f32")])
@pytest.mark.parametrize("lowest", [-np.inf, np.finfo(np.float32).min])
@pytest.mark.parametrize("dup_mode", [0, 1])
def test_position_tables_that_mask_keys(C, heads, hidden, dtype, lowest, dup_mode):
    """Rows of 96, 81 and 50 voxels, one set each, and tables of -inf or the lowest float for pairs further apart than 32 cells on either side
    or on both (the first 32 keys of the queries behind them, the last ones of those in front), for 32 to 63 cells (keys 32 to 63 of the last of 96
    queries) and for all pairs but a voxel with itself.  Every query keeps its own key."""
    grid, win, tau = (96, 3, 1), (96, 1, 1), 96
    rng = np.random.Generator(np.random.Philox(91))
    coords = np.array([(0, i, y, 0) for y, n in enumerate((96, 81, 50)) for i in rng.permutation(n)], np.int32)
    x = synth.make_features(92, len(coords), C, dtype)
    w = synth.make_layer_weights(93, C, heads, hidden, win, dtype)
    own = w["rel_bias"]
    d = np.arange(191) - 95                                  # query - key
    om = orc.partition(coords, grid, win, (0, 0, 0), tau, 0)
    assert om["n_sets"] == 3
    cd = dev_coords(coords)
    maps = gpu_maps(cd, grid, win, (0, 0, 0), tau, 1, 0)
    for name, masked in (("first", d > 32), ("last", d < -32), ("near", np.abs(d) > 32), ("middle", (d >= 32) & (d < 64)), ("others", d != 0)):
        w["rel_bias"] = np.where(masked[None, :], np.float32(lowest), own).astype(np.float32)
        print(f"[case] table masks {name} keys with {lowest}, C={C} {dtype} dup={dup_mode}", flush=True)
        y = dsvt.dsvt_set_attention(dsvt.LayerWeights(w, dup_mode), maps, cd, dev_feats(x, dtype))
        torch.cuda.synchronize()
        assert rel_err(y, orc.set_attention(w, om, coords, x, dup_mode)) < TOL[dtype], name


@pytest.mark.parametrize("C,heads,hidden,dtype", [(192, 8, 384, "bf16"), (128, 8, 256, "bf16"), (64, 4, 128, "bf16"), (64, 4, 128, "f32")])
@pytest.mark.parametrize("tau,dup_mode", [(96, 0), (96, 1), (48, 0), (48, 1)])
def test_tiles_of_one_to_six_row_tiles(C, heads, hidden, dtype, tau, dup_mode):
    """A block over one window of 1 to 96 voxels, in one set or two: the projections' last trip has one or two row tiles, and with a
    single row tile half of the wavefronts have no rows in the LayerNorm phases (C = 64: some no output tile of the MLP either).
    (Two sets of 48: the work list of a frame this small gives each its tile, without one a workgroup takes both.)"""
    grid, win = (12, 12, 1), (12, 12, 1)
    rng = np.random.Generator(np.random.Philox(21))
    ws = [synth.make_layer_weights(22 + a, C, heads, hidden, win, dtype) for a in (0, 1)]
    layers = [dsvt.LayerWeights(w, dup_mode) for w in ws]
    for cnt in (1, 15, 16, 17, 32, 33, 48, 49, 64, 65, 80, 81, 96):
        cell = rng.permutation(144)[:cnt]
        coords = np.stack([0 * cell, cell // 12, cell % 12, 0 * cell], 1).astype(np.int32)
        x = synth.make_features(24 + cnt, cnt, C, dtype)
        print(f"[case] one window of {cnt} voxels C={C} {dtype} tau={tau} dup={dup_mode}", flush=True)
        oms = [orc.partition(coords, grid, win, (0, 0, 0), tau, a) for a in (0, 1)]
        ref = orc.block(ws, oms, coords, x, dup_mode)
        cd = dev_coords(coords)
        for tiles in (True, False) if tau <= 64 else (True,):
            y = dsvt.dsvt_block(layers, [gpu_maps(cd, grid, win, (0, 0, 0), tau, 1, a, tiles=tiles) for a in (0, 1)], cd, dev_feats(x, dtype))
            torch.cuda.synchronize()
            assert rel_err(y, ref) < TOL[dtype], (cnt, tiles)


@pytest.mark.parametrize("C,heads,hidden,dtype", [(192, 8, 384, "bf16"), (128, 8, 256, "bf16"), (64, 4, 128, "bf16"), (64, 4, 128, "f32")])
def test_attention_alone_of_one_to_six_row_tiles(C, heads, hidden, dtype):
    """Attention without the rest of a layer over one window of 1 to 96 voxels: its rows leave by row tile (C = 64 bf16: by pairs of them, the
    last one alone), rows that pad the last row tile not at all."""
    grid, win, tau = (12, 12, 1), (12, 12, 1), 96
    rng = np.random.Generator(np.random.Philox(51))
    w = synth.make_layer_weights(52, C, heads, hidden, win, dtype)
    layer = dsvt.LayerWeights(w)
    for cnt in (1, 15, 16, 17, 31, 32, 33, 48, 49, 64, 65, 80, 81, 95, 96):
        cell = rng.permutation(144)[:cnt]
        coords = np.stack([0 * cell, cell // 12, cell % 12, 0 * cell], 1).astype(np.int32)
        x = synth.make_features(54 + cnt, cnt, C, dtype)
        print(f"[case] attention alone, one window of {cnt} voxels C={C} {dtype}", flush=True)
        om = orc.partition(coords, grid, win, (0, 0, 0), tau, 0)
        cd = dev_coords(coords)
        both = torch.full((cnt + 16, C), 7.0, dtype=layer.dtype, device="cuda")          # (rows past the last one keep what they held)
        y = dsvt.dsvt_set_attention(layer, gpu_maps(cd, grid, win, (0, 0, 0), tau, 1, 0), cd, dev_feats(x, dtype), y=both[:cnt])
        torch.cuda.synchronize()
        assert rel_err(y, orc.set_attention(w, om, coords, x)) < TOL[dtype] and bool((both[cnt:] == 7.0).all()), cnt


def test_position_table_of_more_than_2_gib():
    """A window whose table of relative positions has byte offsets past 2^31 (811 x 811 x 103 entries of eight heads): pairs of voxels whose
    coordinate difference lies at the table's start, in its middle, around 2^31 and at its end."""
    C, heads, win, tau = 128, 8, (406, 406, 52), 32
    far = [(0, 0, 0), (1, 7, 50), (398, 400, 3), (399, 0, 0), (400, 1, 51), (405, 405, 51), (200, 203, 26), (405, 0, 0), (0, 405, 51), (201, 3, 1)]
    coords = np.array([(0, *c) for c in far], np.int32)
    x = synth.make_features(61, len(coords), C, "bf16")
    w = synth.make_layer_weights(62, C, heads, 256, win, "bf16", rel_bias=False)
    size = (2 * win[0] - 1) * (2 * win[1] - 1) * (2 * win[2] - 1)
    at = np.unique(orc.rel_index(coords[:, None, 1:].astype(np.int64), coords[None, :, 1:].astype(np.int64), win))
    assert at[0] == 0 and at[-1] == size - 1 and 10 < np.count_nonzero(at * heads * 4 >= 2 ** 31) < len(at) // 2
    values = np.random.Generator(np.random.Philox(63)).standard_normal((heads, len(at))).astype(np.float32)
    table, table64 = np.zeros((heads, size), np.float32), np.zeros((heads, size))          # (pages nobody writes take no memory)
    table[:, at], table64[:, at] = values, values
    print(f"[case] position table of {table.nbytes} bytes", flush=True)
    om = orc.partition(coords, win, win, (0, 0, 0), tau, 0)
    cd = dev_coords(coords)
    layer = dsvt.LayerWeights(dict(w, rel_bias=table))
    y = dsvt.dsvt_set_attention(layer, gpu_maps(cd, win, win, (0, 0, 0), tau, 1, 0, tiles=False), cd, dev_feats(x, "bf16"))
    torch.cuda.synchronize()
    assert rel_err(y, orc.set_attention(dict(w, rel_bias=table64), om, coords, x)) < TOL["bf16"]


def _windows_of_one_set_and_two(n):
    """n voxels in 24 x 24 windows of 20 to 73 on a 480 x 480 grid."""
    rng = np.random.Generator(np.random.Philox(15))
    cnt, left = [], n
    while left > 0:                                          # windows of one set (up to tau) and of two
        cnt.append(min(left, (48, 49, 50, 51, 60, 64, 65, 72, 73, 20)[len(cnt) % 10]))
        left -= cnt[-1]
    rows = []
    for w, k in enumerate(cnt):
        cell = rng.permutation(576)[:k]
        rows.append(np.stack([0 * cell, 24 * (w // 20) + cell // 24, 24 * (w % 20) + cell % 24, 0 * cell], 1))
    return np.concatenate(rows).astype(np.int32)


@pytest.mark.parametrize("tau,n,dup_mode", [(50, 12288, 0), (50, 12289, 0), (50, 12289, 1), (64, 13568, 1), (64, 13569, 0), (64, 13569, 1),
                                            (72, 15361, 0), (72, 15361, 1), (73, 15617, 0)])
def test_large_sets_around_the_slim_kernel(tau, n, dup_mode):
    """C = 64 in bf16: the frame sizes and set sizes between which the kernel of fewer registers is taken, and full
    windows of 49 to 72 voxels in it (without a tile list too, where a set may have 64)."""
    grid, win, C = (480, 480, 1), (24, 24, 1), 64
    coords = _windows_of_one_set_and_two(n)
    x = synth.make_features(16, n, C, "bf16")
    w = synth.make_layer_weights(17, C, 4, 128, win, "bf16")
    print(f"[case] slim kernel tau={tau} n={n} dup={dup_mode}", flush=True)
    om = orc.partition(coords, grid, win, (0, 0, 0), tau, 0)
    ref = orc.set_attention(w, om, coords, x, dup_mode)
    cd = dev_coords(coords)
    for tiles in (True, False) if tau <= 64 else (True,):
        maps = gpu_maps(cd, grid, win, (0, 0, 0), tau, 1, 0, tiles=tiles)
        y = dsvt.dsvt_set_attention(dsvt.LayerWeights(w, dup_mode), maps, cd, dev_feats(x, "bf16"))
        torch.cuda.synchronize()
        assert rel_err(y, ref) < TOL["bf16"]


@pytest.mark.parametrize("tau,n", [(50, 12288), (50, 12289), (64, 13568), (64, 13569), (72, 15360), (72, 15361), (73, 15617)])
@pytest.mark.parametrize("dup_mode", [0, 1])
def test_block_around_the_slim_kernel(tau, n, dup_mode):
    """The same lines with the whole layer behind the attention: residuals, LayerNorms and MLP, twice."""
    grid, win, C = (480, 480, 1), (24, 24, 1), 64
    coords = _windows_of_one_set_and_two(n)
    x = synth.make_features(18, n, C, "bf16")
    ws = [synth.make_layer_weights(19 + a, C, 4, 128, win, "bf16") for a in (0, 1)]
    print(f"[case] block, slim kernel tau={tau} n={n} dup={dup_mode}", flush=True)
    oms = [orc.partition(coords, grid, win, (0, 0, 0), tau, a) for a in (0, 1)]
    ref = orc.block(ws, oms, coords, x, dup_mode)
    layers, cd = [dsvt.LayerWeights(w, dup_mode) for w in ws], dev_coords(coords)
    for tiles in (True, False) if tau <= 64 else (True,):
        y = dsvt.dsvt_block(layers, [gpu_maps(cd, grid, win, (0, 0, 0), tau, 1, a, tiles=tiles) for a in (0, 1)], cd, dev_feats(x, "bf16"))
        torch.cuda.synchronize()
        assert rel_err(y, ref) < TOL["bf16"], tiles


@pytest.mark.parametrize("C,heads,hidden,dtype", [(192, 8, 384, "bf16"), (128, 8, 256, "bf16"), (64, 4, 128, "bf16"), (64, 4, 128, "f32")])
@pytest.mark.parametrize("tau,dup_mode", [(96, 0), (72, 1), (48, 0), (36, 0), (36, 1)])
def test_workgroups_that_take_several_tiles(C, heads, hidden, dtype, tau, dup_mode):
    """Frames of one tile per workgroup (256 of them, 512 at C = 64 bf16), of one less and one more, of two, of two and one, and so on: a
    workgroup's next tile is fetched during the one before, its rows over that one's queries.  The windows are five patterns in turn, so five
    windows' oracle gives every row.  Sets of more than 48 voxels have a tile each; of the smaller ones as many windows are taken as make
    the tiles that are wanted."""
    win, sizes = (12, 12, 1), [min(s, 144) for s in (tau, tau - 1, tau // 2 + 1, tau - 3, tau // 2 + 2)]
    windows_tiles = {36: ((311, 255), (380, 256), (555, 257), (1105, 511), (1106, 512), (1600, 647), (3054, 1024), (3057, 1025)),
                     48: ((255, 255), (333, 256), (334, 257), (664, 511), (665, 512), (1000, 600), (1706, 1024), (2041, 1025), (3061, 1537))}
    windows_tiles = windows_tiles.get(tau, [(n, n) for n in (255, 256, 257, 511, 512, 513, 1024, 1025, 1537)])
    rng = np.random.Generator(np.random.Philox(31))
    cells = [rng.permutation(144)[:s] for s in sizes]
    place = lambda w, cell: np.stack([0 * cell, 12 * (w // 60) + cell // 12, 12 * (w % 60) + cell % 12, 0 * cell], 1).astype(np.int32)
    ws = [synth.make_layer_weights(32 + a, C, heads, hidden, win, dtype) for a in (0, 1)]
    layers = [dsvt.LayerWeights(w, dup_mode) for w in ws]
    one = np.concatenate([place(k, c) for k, c in enumerate(cells)])
    x1 = synth.make_features(34, len(one), C, dtype)
    ref1 = orc.block(ws, [orc.partition(one, (720, 720, 1), win, (0, 0, 0), tau, a) for a in (0, 1)], one, x1, dup_mode)
    att1 = orc.set_attention(ws[0], orc.partition(one, (720, 720, 1), win, (0, 0, 0), tau, 0), one, x1, dup_mode)
    first = np.cumsum([0] + sizes)
    for n_win, n_tiles in windows_tiles:
        coords = np.concatenate([place(w, cells[w % 5]) for w in range(n_win)])
        rows = np.concatenate([np.arange(first[w % 5], first[w % 5 + 1]) for w in range(n_win)])
        cd, xd = dev_coords(coords), dev_feats(x1[rows], dtype)
        maps = [gpu_maps(cd, (720, 720, 1), win, (0, 0, 0), tau, 1, a) for a in (0, 1)]
        print(f"[case] {n_win} windows, {int(maps[0].n_tiles.item())} tiles, C={C} {dtype} tau={tau} dup={dup_mode}", flush=True)
        assert [int(m.n_tiles.item()) for m in maps] == [n_tiles, n_tiles]
        y = dsvt.dsvt_block(layers, maps, cd, xd)
        z = dsvt.dsvt_set_attention(layers[0], maps[0], cd, xd)
        torch.cuda.synchronize()
        assert rel_err(y, ref1[rows]) < TOL[dtype] and rel_err(z, att1[rows]) < TOL[dtype]
        again = dsvt.dsvt_block(layers, maps, cd, xd, x_out=xd)                  # in place: the same bits
        torch.cuda.synchronize()
        assert torch.equal(again, y)


@pytest.mark.parametrize("C,heads,hidden,dtype,n_win", [(192, 8, 384, "bf16", 2600), (192, 8, 384, "bf16", 3413), (128, 8, 256, "bf16", 2901),
                                                        (64, 4, 128, "bf16", 5003), (64, 4, 128, "f32", 2701)])
@pytest.mark.parametrize("dup_mode", [0, 1])
def test_frames_of_several_rounds_and_a_part(C, heads, hidden, dtype, n_win, dup_mode):
    """Frames of more than two rounds of tiles, the last of them partial, of windows of 1 to 36 voxels in random order: which workgroups take
    a tile more, and which ones, depends on the tiles' rows; every tile is to be done once.  Five windows' oracle gives every row.  A work
    list that ends early (128 tiles fewer, then fewer than there are workgroups) leaves the rows of the tiles past its end alone."""
    win, tau, sizes = (12, 12, 1), 36, (36, 31, 22, 17, 1)
    rng = np.random.Generator(np.random.Philox(81))
    cells = [rng.permutation(144)[:s] for s in sizes]
    which = rng.choice(5, n_win, p=(0.35, 0.2, 0.2, 0.2, 0.05))
    place = lambda w, cell: np.stack([0 * cell, 12 * (w // 72) + cell // 12, 12 * (w % 72) + cell % 12, 0 * cell], 1).astype(np.int32)
    grid = (864, 864, 1)
    ws = [synth.make_layer_weights(82 + a, C, heads, hidden, win, dtype) for a in (0, 1)]
    layers = [dsvt.LayerWeights(w, dup_mode) for w in ws]
    one = np.concatenate([place(k, c) for k, c in enumerate(cells)])
    x1 = synth.make_features(84, len(one), C, dtype)
    ref1 = orc.block(ws, [orc.partition(one, grid, win, (0, 0, 0), tau, a) for a in (0, 1)], one, x1, dup_mode)
    first = np.cumsum((0,) + sizes)
    coords = np.concatenate([place(w, cells[k]) for w, k in enumerate(which)])
    rows = np.concatenate([np.arange(first[k], first[k + 1]) for k in which])
    cd, xd = dev_coords(coords), dev_feats(x1[rows], dtype)
    maps = [gpu_maps(cd, grid, win, (0, 0, 0), tau, 1, a) for a in (0, 1)]
    n_tiles, groups = int(maps[0].n_tiles.item()), 512 if (C, dtype) == (64, "bf16") else 256
    print(f"[case] {n_win} windows, {len(coords)} voxels, {n_tiles} tiles, C={C} {dtype} dup={dup_mode}", flush=True)
    assert len(coords) > 96 * 2 * groups and n_tiles > 2 * groups and n_tiles % groups != 0
    y = dsvt.dsvt_block(layers, maps, cd, xd)
    torch.cuda.synchronize()
    assert rel_err(y, ref1[rows]) < TOL[dtype]
    for keep in (n_tiles - 128, groups - 1):
        out = torch.full_like(xd, 7.0)
        for m in maps:
            m.n_tiles.fill_(keep)
        dsvt.dsvt_block(layers, maps, cd, xd, x_out=out)
        torch.cuda.synchronize()
        done = np.zeros(len(coords), bool)
        desc = maps[0].tile_desc[:keep].cpu().numpy()
        listed = desc[:, 64::2][:, :96]
        done[listed[(np.arange(96)[None, :] < desc[:, :1]) & (listed >= 0)]] = True
        assert 0 < done.sum() < len(coords) and bool((out[torch.as_tensor(~done).cuda()] == 7.0).all())
        assert torch.equal(out[torch.as_tensor(done).cuda()], y[torch.as_tensor(done).cuda()])


@pytest.mark.parametrize("C,heads,hidden,dtype,n_win", [(192, 8, 384, "bf16", 2600), (128, 8, 256, "bf16", 2600), (64, 4, 128, "bf16", 5003), (64, 4, 128, "f32", 2600)])
def test_work_lists_of_whole_rounds_and_a_tile_more_or_less(C, heads, hidden, dtype, n_win):
    """The kernel for frames of several rounds with lists of exactly one and two rounds (every workgroup has the same number of tiles), of a tile
    more than one (nobody has a second one but its taker) and of a tile less than two: each listed tile is done, with the bits that the whole list gives it, and
    no other row is written."""
    win, tau, grid = (12, 12, 1), 36, (864, 864, 1)
    rng = np.random.Generator(np.random.Philox(121))
    sizes = rng.choice((36, 31, 22, 17), n_win)
    cells = [rng.permutation(144)[:k] for k in sizes]
    coords = np.concatenate([np.stack([0 * c, 12 * (w // 72) + c // 12, 12 * (w % 72) + c % 12, 0 * c], 1) for w, c in enumerate(cells)]).astype(np.int32)
    layers = [dsvt.LayerWeights(synth.make_layer_weights(122 + a, C, heads, hidden, win, dtype)) for a in (0, 1)]
    cd, xd = dev_coords(coords), dev_feats(synth.make_features(124, len(coords), C, dtype), dtype)
    maps = [gpu_maps(cd, grid, win, (0, 0, 0), tau, 1, a) for a in (0, 1)]
    n_tiles, groups = int(maps[0].n_tiles.item()), 512 if (C, dtype) == (64, "bf16") else 256
    assert len(coords) > 96 * 2 * groups and n_tiles > 2 * groups
    y = dsvt.dsvt_block(layers, maps, cd, xd)
    desc = maps[0].tile_desc.cpu().numpy().reshape(-1, 256)
    for keep in (groups, groups + 1, 2 * groups - 1, 2 * groups):
        print(f"[case] {keep} of {n_tiles} tiles, C={C} {dtype}", flush=True)
        out = torch.full_like(xd, 7.0)
        for m in maps:
            m.n_tiles.fill_(keep)
        dsvt.dsvt_block(layers, maps, cd, xd, x_out=out)
        torch.cuda.synchronize()
        done = np.zeros(len(coords), bool)
        listed = desc[:keep, 64::2][:, :96]
        done[listed[(np.arange(96)[None, :] < desc[:keep, :1]) & (listed >= 0)]] = True
        done = torch.as_tensor(done).cuda()
        assert 0 < int(done.sum()) < len(coords) and bool((out[~done] == 7.0).all()) and torch.equal(out[done], y[done]), keep


@pytest.mark.parametrize("C,heads,hidden,dtype", [(128, 8, 256, "bf16"), (64, 4, 128, "bf16"), (64, 4, 128, "f32")])
@pytest.mark.parametrize("dup_mode", [0, 1])
def test_attention_items_split_and_whole(C, heads, hidden, dtype, dup_mode):
    """Tiles of few attention items split them (C = 64 bf16: up to 256 tiles, sets of one and two key tiles); a head's result does not
    depend on it.  Without a work list a tile is two sets: 512 windows are 256 tiles, 514 are 257."""
    win, sizes = (12, 12, 1), (16, 17, 32, 1, 33, 5, 48, 48, 9, 12)
    rng = np.random.Generator(np.random.Philox(41))
    cells = [rng.permutation(144)[:s] for s in sizes]
    place = lambda w: np.stack([0 * cells[w % 10], 12 * (w // 50) + cells[w % 10] // 12, 12 * (w % 50) + cells[w % 10] % 12, 0 * cells[w % 10]], 1)
    coords = np.concatenate([place(w) for w in range(514)]).astype(np.int32)
    first = sum(sizes[w % 10] for w in range(512))
    w, x = synth.make_layer_weights(42, C, heads, hidden, win, dtype), synth.make_features(43, len(coords), C, dtype)
    layer = dsvt.LayerWeights(w, dup_mode)
    out = []
    for n in (first, len(coords)):
        cd = dev_coords(coords[:n])
        maps = gpu_maps(cd, (600, 600, 1), win, (0, 0, 0), 48, 1, 0, tiles=False)
        print(f"[case] items split and whole C={C} {dtype} dup={dup_mode} {int(maps.n_sets.item())} sets", flush=True)
        assert int(maps.n_sets.item()) == (512 if n == first else 514)
        out.append(dsvt.dsvt_set_attention(layer, maps, cd, dev_feats(x[:n], dtype)))
    torch.cuda.synchronize()
    assert torch.equal(out[0], out[1][:first])
    om = orc.partition(coords, (600, 600, 1), win, (0, 0, 0), 48, 0)
    assert rel_err(out[1], orc.set_attention(w, om, coords, x, dup_mode)) < TOL[dtype]


@pytest.mark.parametrize("C,heads,hidden,dtype", [(192, 8, 384, "bf16"), (128, 8, 256, "bf16"), (64, 4, 128, "bf16"), (64, 4, 128, "f32")])
@pytest.mark.parametrize("dup_mode", [0, 1])
def test_a_set_alone_in_its_tile_and_beside_another(C, heads, hidden, dtype, dup_mode):
    """A set of one or two key tiles that has its tile to itself is split into items of a quarter of the heads, beside another of two key tiles
    it is not: the same bits.  Without a work list a tile is two sets."""
    grid, win, tau = (12, 24, 1), (12, 12, 1), 48
    rng = np.random.Generator(np.random.Philox(101))
    w = synth.make_layer_weights(102, C, heads, hidden, win, dtype)
    layer = dsvt.LayerWeights(w, dup_mode)
    for cnt in (7, 16, 17, 25, 32):
        cells = [rng.permutation(144)[:n] for n in (cnt, 32)]
        coords = np.concatenate([np.stack([0 * c, c // 12, 12 * k + c % 12, 0 * c], 1) for k, c in enumerate(cells)]).astype(np.int32)
        x = synth.make_features(103 + cnt, len(coords), C, dtype)
        print(f"[case] {cnt} voxels alone and beside 32, C={C} {dtype} dup={dup_mode}", flush=True)
        out = []
        for n in (cnt, len(coords)):
            cd = dev_coords(coords[:n])
            maps = gpu_maps(cd, grid, win, (0, 0, 0), tau, 1, 0, tiles=False)
            assert int(maps.n_sets.item()) == (1 if n == cnt else 2)
            out.append(dsvt.dsvt_set_attention(layer, maps, cd, dev_feats(x[:n], dtype)))
        torch.cuda.synchronize()
        assert torch.equal(out[0], out[1][:cnt]), cnt


@pytest.mark.parametrize("C,heads,hidden", [(192, 8, 384), (128, 8, 256), (64, 4, 128)])
@pytest.mark.parametrize("tau,cnt", [(48, 48), (48, 32), (96, 96), (96, 70)])
@pytest.mark.parametrize("dup_mode", [0, 1])
def test_sums_of_probabilities_are_of_32_bit_terms(C, heads, hidden, tau, cnt, dup_mode):
    """bf16, small and large sets, without and with doubled voxels. All keys but the query's own have one probability, in the
    middle between two bf16 numbers but for 2^-12 of it, and only the first voxel has values: its output is the value over the sum.  The value's
    and the output's rounding are at most 2^-9 each way and even out over all mantissas and both directions of the probability
    (mean of C: below 2^-11, five times its deviation for 64); probabilities rounded in front of the sum move it by up to 2^-8."""
    grid, win = (96, 1, 1), (96, 1, 1)
    coords = np.array([(0, i, 0, 0) for i in range(cnt)], np.int32)
    x = np.zeros((cnt, C), np.float32)
    x[0] = 1.0 + np.arange(C) % 128 / 128.0
    w = synth.make_layer_weights(111, C, heads, hidden, win, "bf16")
    w["w_qkv"] = np.concatenate([np.zeros((2 * C, C)), np.eye(C)]).astype(np.float32)
    w["w_o"], w["b_qkv"], w["b_o"] = np.eye(C, dtype=np.float32), np.zeros(3 * C, np.float32), np.zeros(C, np.float32)
    om = orc.partition(coords, grid, win, (0, 0, 0), tau, 0)
    cd = dev_coords(coords)
    maps = gpu_maps(cd, grid, win, (0, 0, 0), tau, 1, 0)
    for p in (1 + 2.0 ** -8 - 2.0 ** -12, 1 + 2.0 ** -8 + 2.0 ** -12):
        w["rel_bias"] = np.where(np.arange(191)[None, :] == 95, 0.0, np.log(p / 2)).repeat(heads, 0).astype(np.float32)
        print(f"[case] probabilities of {p} / 2, C={C} tau={tau} {cnt} voxels dup={dup_mode}", flush=True)
        y = dsvt.dsvt_set_attention(dsvt.LayerWeights(w, dup_mode), maps, cd, dev_feats(x, "bf16"))
        torch.cuda.synchronize()
        ref = orc.set_attention(w, om, coords, x, dup_mode)[0]
        assert abs(np.mean(y[0].double().cpu().numpy() / ref) - 1) < 2.0 ** -11, p


@pytest.mark.parametrize("C,heads,dtype", [(192, 8, "bf16"), (128, 8, "bf16"), (64, 4, "bf16"), (64, 4, "f32")])
@pytest.mark.parametrize("n_multi,n_single", [(0, 24576), (0, 24577), (1, 24623), (8193, 9000), (12289, 0), (20, 24576 + 47)])
def test_pool_regions_of_one_voxel_apart(C, heads, dtype, n_multi, n_single):
    """Frames above and around the size from which regions of one voxel are taken apart: only such regions, none,
    a remainder of either kind; with the scratch the size call names and with the plain layout's, the same result.
    A call at that size (24,576 voxels) asks for the plain layout only."""
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
    assert sizes[0] > sizes[1] if n > 24576 else sizes[0] == sizes[1]
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


def _pool_frame(rng, grid, pool, batch, sizes, outside, repeats):
    """A frame of regions of the given numbers of voxels (full regions only where the grid cuts none short), then cells outside
    the grid and repeats: coords, the features' index of every row, and the rows that count (each cell once)."""
    full = [g // p for g, p in zip(grid, pool)]
    P = int(np.prod(pool))
    reg = rng.permutation(batch * int(np.prod(full)))[:len(sizes)]
    slot = np.argsort(rng.random((len(sizes), P)), 1)
    k, j = np.nonzero(np.arange(P)[None, :] < np.asarray(sizes)[:, None])
    s, r = slot[k, j], reg[k]
    cells = np.stack([r // int(np.prod(full)), r // (full[1] * full[2]) % full[0] * pool[0] + s // (pool[1] * pool[2]),
                      r // full[2] % full[1] * pool[1] + s // pool[2] % pool[1], r % full[2] * pool[2] + s % pool[2]], 1)
    if any(g % p for g, p in zip(grid, pool)):               # the regions cut short: the grid's last cell of every frame
        cells = np.concatenate([cells, [[b] + [g - 1 for g in grid] for b in range(batch)]])
    n = len(cells)
    bad = np.tile(cells[:1], (outside, 1))
    bad[:, 1:] = rng.integers(0, 2, (outside, 3)) * (np.array(grid) + 1) - 1
    bad[:, 0] = rng.integers(-1, batch + 1, outside)
    bad[:, 1] = np.where(bad[:, 1] < 0, bad[:, 1], grid[0])
    rep = rng.integers(0, n, repeats)
    feat = np.concatenate([np.arange(n), n + np.arange(outside), rep])
    order = rng.permutation(n + outside + repeats)
    return np.concatenate([cells, bad, cells[rep]])[order].astype(np.int32), feat[order], n


def _cycle(values, total):
    out = []
    while total > 0:
        out.append(min(values[len(out) % len(values)], total))
        total -= out[-1]
    return out


@pytest.mark.parametrize("C,heads,dtype,grid,pool,batch,sizes,outside,repeats", [
    (192, 8, "bf16", (100, 90, 9), (2, 2, 2), 2, _cycle((1, 1, 8, 1, 7, 2, 1, 1, 5), 26000), 0, 0),           # one in two alone, up to eight
    (64, 4, "f32", (101, 91, 9), (2, 2, 2), 2, _cycle((1, 1, 2, 1, 3, 1), 25000), 300, 400),
    (64, 4, "bf16", (128, 128, 8), (1, 1, 2), 1, _cycle((1, 2), 25001), 0, 77),
    (128, 8, "bf16", (200, 130, 1), (1, 1, 1), 1, [1] * 25001, 5, 9),                                       # a repeated cell is a region of two
    (64, 4, "f32", (128, 128, 8), (2, 2, 1), 1, _cycle((4, 4, 4, 1), 30000), 0, 0),                           # kept together: one in four alone
    (192, 8, "bf16", (128, 128, 8), (2, 2, 2), 1, _cycle((8, 8, 1), 40000), 100, 0),                          # together, five passes and more
    (64, 4, "bf16", (128, 128, 8), (1, 1, 4), 1, [1] * 10000 + [3] * 15000, 0, 0),                            # together: two fifths alone
    (64, 4, "bf16", (128, 128, 8), (1, 1, 4), 1, [1] * 10001 + [3] * 15000, 0, 0),                            # apart: one more
    (64, 4, "f32", (160, 160, 8), (1, 1, 4), 1, [1] * 20000 + [4] * 31000, 0, 0),                             # together: 20,000 alone
    (64, 4, "f32", (160, 160, 8), (1, 1, 4), 1, [1] * 20001 + [4] * 31000, 0, 0),                             # apart: one more
    (64, 4, "bf16", (128, 128, 8), (1, 1, 4), 1, [1] * 5000 + [2] * 10000, 0, 0),                             # apart: under two voxels a region
    (64, 4, "bf16", (4096, 4096, 2), (1, 1, 2), 1, _cycle((1, 2, 1), 25000), 0, 0),                            # larger layout past the built-in scratch
    (64, 4, "f32", (128, 128, 8), (1, 1, 4), 1, [], 25000, 0)])                                              # nothing inside the grid
def test_pool_apart_over_region_forms(C, heads, dtype, grid, pool, batch, sizes, outside, repeats):
    """The large frames' path over regions of one to eight cells, two frames, grids that cut regions short, cells outside the
    grid and repeated ones, at the lines between regions kept together and apart; with the smaller scratch and
    on the built-in one too (where the larger layout fits it and where it does not), the same rows."""
    rng = np.random.Generator(np.random.Philox(25))
    coords, feat, n = _pool_frame(rng, grid, pool, batch, sizes, outside, repeats) if sizes else (
        np.tile(np.array([[0, -1, 0, 0]], np.int32), (outside, 1)), np.arange(outside), 0)
    x_all = synth.make_features(26, max(n + outside, 1), C, dtype)
    x, N = x_all[feat], len(coords)
    w = synth.make_pool_weights(27, C, heads, dtype)
    print(f"[case] pool forms C={C} {dtype} {pool} batch {batch}, {N} rows, {n} cells", flush=True)
    assert N > 24576
    once = np.zeros(N, bool)
    once[np.unique(feat, return_index=True)[1]] = True
    once &= feat < n
    ref_c, ref = orc.attn_pool(w, coords[once], x[once], grid, pool, 1) if n else (np.zeros((0, 4), np.int32), np.zeros((0, C)))
    pw, plain = dsvt.PoolWeights(w, grid, pool, batch, 1), dsvt.PoolWeights(w, grid, pool, batch, 0)
    cd, xd = dev_coords(coords), dev_feats(x, dtype)
    for way in (dsvt.dsvt_attn_pool_workspace_size(pw, N), dsvt.dsvt_attn_pool_workspace_size(plain, N), "static", "static"):
        out = (torch.full((N, 4), -7, dtype=torch.int32, device="cuda"), torch.zeros_like(xd),
               torch.zeros(1, dtype=torch.int32, device="cuda"), torch.zeros(1, dtype=torch.int32, device="cuda"))
        if way == "static":
            dsvt.dsvt_attn_pool_static(pw, cd, xd, out)
        else:
            dsvt.dsvt_attn_pool(pw, cd, xd, out=out, ws=torch.full((way,), 0x5A, dtype=torch.uint8, device="cuda"))
        torch.cuda.synchronize()
        assert int(out[3].item()) == (dsvt.binding.ST_COORD_RANGE if outside else 0)
        m = int(out[2].item())
        assert m == len(ref_c) and np.array_equal(out[0][:m].cpu().numpy(), ref_c)
        assert torch.all(out[0][m:] == -7) and torch.all(out[1][m:] == 0)
        if m:
            assert rel_err(out[1][:m], ref) < TOL[dtype]


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


def _vfe_plain_scratch(cells, n_points, max_voxels, f_in):
    """Scratch of a call that counts its points by voxel: byte map, bitmap and its prefix, counts and their prefix, three
    words and a run descriptor per point, the row count, the sorted rows."""
    words = -(-(-(-cells // 32)) // 64) * 64
    parts = [32 * words, 4 * words, 4 * words, 4 * (max_voxels + 1), 4 * (max_voxels + 1)] + [4 * n_points] * 3
    return sum(-(-p // 256) * 256 for p in parts + [16 * n_points, 4, n_points * -(-f_in // 4) * 16])


@pytest.mark.parametrize("grid,batch,n_points,f_in,cap,ways", [
    # both ways, the scratch choosing: 64 words exactly (the last cell's run ends behind the last word), a part of the voxels
    ((64, 64, 1), 1, 1500, 5, 500, 2), ((64, 64, 4), 1, 3000, 5, None, 2), ((64, 64, 4), 1, 3000, 5, 700, 2),
    ((61, 59, 3), 2, 2500, 3, 1000, 2), ((33, 31, 3), 2, 700, 16, 1, 2), ((512, 512, 2), 1, 3000, 6, None, 2),  # 16,384 words: one scan chunk
    ((520, 512, 2), 1, 3000, 12, 2000, 2),
    # by cell only: its layout is the smaller one
    ((64, 32, 1), 1, 5000, 5, None, 1), ((64, 32, 1), 1, 5000, 5, 700, 1), ((33, 31, 3), 2, 4000, 3, 1000, 1),
    ((1, 1, 1), 1, 257, 4, None, 2),
    # around the lines between them: 1.5 M cells + 20 a point, 80,000 points, 8 M cells
    ((1000, 1520, 1), 1, 1000, 5, None, 2), ((1000, 1521, 1), 1, 1000, 5, None, 0), ((1000, 1521, 1), 1, 1000, 5, 500, 0),
    ((256, 256, 128), 1, 80000, 4, None, 2), ((256, 256, 128), 1, 79999, 4, 40000, 0), ((256, 256, 129), 1, 80000, 4, 50000, 0),
    ((256, 256, 128), 1, 2000, 5, None, 0), ((256, 256, 129), 1, 2000, 5, None, 0)])
def test_vfe_counting_by_cell_and_by_voxel(grid, batch, n_points, f_in, cap, ways):
    """Both ways of counting: voxels, their order, the maxima and the overflow report are the oracle's bit for bit; every
    corner of the grid is occupied, and points lie outside it.  ways: 2 = the call prefers to count by cell and counts
    by voxel in the smaller scratch, 1 = it has no need of more than that scratch, 0 = it prefers to count by voxel."""
    lo, size = (-4.0, -2.0, -1.0), (0.5, 0.25, 0.125)
    rng = np.random.Generator(np.random.Philox(41))
    ext = np.array(grid, np.float64) * size
    pts = rng.random((n_points, f_in)).astype(np.float32)
    pts[:, :3] = lo + ext * (1.1 * rng.random((n_points, 3)) - 0.05)
    for k in range(8):
        pts[k, :3] = [l + s * (0.5 if not k >> a & 1 else g - 0.5) for a, (l, s, g) in enumerate(zip(lo, size, grid))]
    pts[8, 0] = np.nan
    pb = rng.integers(0, batch, n_points).astype(np.int32)
    pb[:8] = batch - 1
    rc, rx = orc.voxel_max_vfe(pts, pb, lo, size, grid, batch)
    assert cap is None or cap < len(rc)
    cap = cap or len(rc)
    kept = min(cap, len(rc))
    print(f"[case] vfe by cell / by voxel grid={grid} batch={batch} points={n_points} cap={cap} of {len(rc)}", flush=True)
    vfe = dsvt.Vfe(grid, batch, lo, size, f_in, f_in, "f32", n_points, cap)
    cells, plain = batch * grid[0] * grid[1] * grid[2], _vfe_plain_scratch(batch * grid[0] * grid[1] * grid[2], n_points, cap, f_in)
    own = vfe.ws.numel()
    assert own > plain if ways == 2 else own == plain
    for nbytes in (own, plain, own + 64 * cells):
        vfe.ws = torch.full((nbytes,), 0x5A, dtype=torch.uint8, device="cuda")
        vfe.x.fill_(-7.0), vfe.coords.fill_(-7), vfe.status.zero_()
        dsvt.dsvt_vfe(vfe, torch.as_tensor(pts).cuda(), torch.as_tensor(pb).cuda())
        torch.cuda.synchronize()
        assert int(vfe.n_voxels.item()) == len(rc)
        assert int(vfe.status.item()) == (dsvt.binding.ST_VOXEL_OVERFLOW if cap < len(rc) else 0)
        assert np.array_equal(vfe.coords[:kept].cpu().numpy(), rc[:kept])
        assert np.array_equal(vfe.x[:kept].double().cpu().numpy(), rx[:kept])


@pytest.mark.parametrize("C,f_in,dt", [(1, 5, "f32"), (100, 3, "f32"), (64, 7, "f32"), (192, 5, "bf16"), (260, 4, "f32")])
@pytest.mark.parametrize("bias", [False, True])
def test_vfe_runs_at_the_staging_edges(C, f_in, dt, bias):
    """Voxels whose points end at, before and behind a wavefront's rows, its first load and its staged rows; channels that
    do not fill the lanes, rows that do not fill the kernel's row length, no bias."""
    counts = (1, 15, 16, 17, 47, 63, 64, 65, 1, 1, 127, 128, 129, 143, 144, 300, 1, 2, 16, 16)
    rng = np.random.Generator(np.random.Philox(51))
    cell = np.repeat(np.arange(len(counts)), counts)[rng.permutation(sum(counts))]
    pts = rng.random((len(cell), f_in)).astype(np.float32)
    pts[:, 0] = cell + 0.5 * pts[:, 0] + 0.25
    pb = np.zeros(len(cell), np.int32)
    grid, lo, size = (len(counts), 1, 1), (0.0, 0.0, 0.0), (1.0, 1.0, 1.0)
    w, b = synth.make_vfe_weights(52, C, f_in)
    print(f"[case] vfe runs C={C} f_in={f_in} {dt} bias={bias}", flush=True)
    rc, rx = orc.voxel_max_vfe(pts, pb, lo, size, grid, 1, w, b if bias else np.zeros_like(b), False)
    vfe = dsvt.Vfe(grid, 1, lo, size, f_in, C, dt, len(pts), len(pts), torch.as_tensor(w).cuda(),
                   torch.as_tensor(b).cuda() if bias else None, False)
    dsvt.dsvt_vfe(vfe, torch.as_tensor(pts).cuda(), None)
    torch.cuda.synchronize()
    n = int(vfe.n_voxels.item())
    assert n == len(rc) and np.array_equal(vfe.coords[:n].cpu().numpy(), rc)
    assert rel_err(vfe.x[:n], rx) <= (1e-5 if dt == "f32" else 4e-3)        # f_in fused products; one rounding to bf16
