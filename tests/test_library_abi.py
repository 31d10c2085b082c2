"""The C-ABI library loads and exports every function include/dsvt.h declares (no compute calls)."""
import ctypes
import os
import re

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
LIB = os.path.join(ROOT, "paper_2301_06051_amd", "libdsvt.so")


def _declared():
    text = open(os.path.join(ROOT, "include", "dsvt.h")).read()
    text = re.sub(r"/\*.*?\*/", "", text, flags=re.S)
    return sorted(set(re.findall(r"\b(dsvt_[a-z_0-9]+)\s*\(", text)))


def test_header_declares_the_four_entry_points():
    names = _declared()
    for must in ("dsvt_partition", "dsvt_set_attention", "dsvt_block", "dsvt_attn_pool"):
        assert must in names


def test_library_exports_every_declared_symbol():
    if not os.path.exists(LIB):
        import __graft_entry__
        __graft_entry__.build()
    lib = ctypes.CDLL(LIB)
    for name in _declared():
        assert hasattr(lib, name), name


def test_library_exports_nothing_the_header_does_not_declare():
    """Every exported dsvt_* function is a declared one: no debug or instrumentation entry points beside the header's."""
    import subprocess
    if not os.path.exists(LIB):
        import __graft_entry__
        __graft_entry__.build()
    out = subprocess.run(["nm", "-D", "--defined-only", LIB], capture_output=True, text=True, check=True).stdout
    exported = {l.split()[-1] for l in out.splitlines() if l.split() and l.split()[-2] in ("T", "t") and l.split()[-1].startswith("dsvt_")}
    assert exported and exported <= set(_declared()), sorted(exported - set(_declared()))


def test_instrumented_library_adds_one_symbol_only():
    """The optional phase-clock build of the layer kernel is the product library plus dsvt_debug_phase_clocks."""
    import subprocess
    from paper_2301_06051_amd.build import PHASE_LIB
    if not os.path.exists(PHASE_LIB):
        pytest.skip("instrumented library not built")
    out = subprocess.run(["nm", "-D", "--defined-only", PHASE_LIB], capture_output=True, text=True, check=True).stdout
    exported = {l.split()[-1] for l in out.splitlines() if l.split() and l.split()[-2] in ("T", "t") and l.split()[-1].startswith("dsvt_")}
    assert exported - set(_declared()) == {"dsvt_debug_phase_clocks"}


def _kernel_metadata(lib):
    """Name, spilled vector registers, scratch bytes per lane and spilled scalar registers of every kernel in the library: the metadata notes of the
    gfx950 code objects in its offload bundles (a table of (offset, size, id length, id) behind a magic text and a count)."""
    import struct
    import subprocess
    import tempfile
    blob, magic, out, at = open(lib, "rb").read(), b"__CLANG_OFFLOAD_BUNDLE__", [], 0
    while (at := blob.find(magic, at)) >= 0:
        pos = at + len(magic) + 8
        for _ in range(struct.unpack_from("<Q", blob, pos - 8)[0]):
            off, size, n = struct.unpack_from("<QQQ", blob, pos)
            target, pos = blob[pos + 24:pos + 24 + n], pos + 24 + n
            if b"gfx950" in target:
                with tempfile.NamedTemporaryFile() as f:
                    f.write(blob[at + off:at + off + size])
                    f.flush()
                    text = subprocess.run(["/opt/rocm/llvm/bin/llvm-readelf", "--notes", f.name], capture_output=True, text=True, check=True).stdout
                for kernel in text.split("  - .agpr_count:")[1:]:
                    field = lambda name: re.search(rf"\.{name}: +(\S+)", kernel).group(1)
                    out.append((field("symbol"), int(field("vgpr_spill_count")), int(field("private_segment_fixed_size")),
                                int(field("sgpr_spill_count"))))
        at = pos
    return out


def test_no_kernel_spills_vector_registers():
    """Scratch reloads wait for every outstanding load, so one spill undoes the layer kernel's early weight requests."""
    if not os.path.exists(LIB):
        pytest.skip("library not built")
    kernels = _kernel_metadata(LIB)
    assert len([k for k in kernels if "k_layer" in k[0]]) == 18 and any("kp_attention" in k[0] for k in kernels)
    assert [k for k in kernels if k[1] or (k[2] and "k_layer" in k[0])] == []


def test_layer_kernel_spills_no_scalar_registers():
    """Every pointer of the arguments kept through the loop over tiles is two lanes of a vector register written and read back: up to 30 a
    kernel, 2-5 % of a layer."""
    if not os.path.exists(LIB):
        pytest.skip("library not built")
    assert [k for k in _kernel_metadata(LIB) if "k_layer" in k[0] and k[3]] == []


@pytest.mark.parametrize("parts,compiles", [(1, True), (2, True), (3, False), (6, False)])
def test_projection_over_parts_of_the_row_tiles_that_it_cannot_cover_does_not_compile(tmp_path, parts, compiles):
    """GemmPhase::run() gives an item all row tiles or a half of them; the phases that take thirds have walks of their own."""
    import subprocess
    from paper_2301_06051_amd import build
    if not os.path.exists(build.HIPCC):
        pytest.skip("no compiler")
    src = tmp_path / "phase.hip"
    src.write_text('#include "mma.h"\n'
                   "__global__ void k(const float* w, const float* b, float* x) {\n"
                   f"  GemmPhase<float, 1, 64, 64, 8, {parts}> phase(w, threadIdx.x >> 6);\n"
                   "  phase.prefetch();\n"
                   "  phase.run(x, 72, 6, b, [&](int o0, int r, f32x4 (&acc)[1]) { x[o0 + r] = acc[0][0]; });\n"
                   "}\n")
    r = subprocess.run([build.HIPCC, *build.FLAGS, "--cuda-device-only", "-fsyntax-only", str(src)], capture_output=True, text=True)
    assert (r.returncode == 0) == compiles, r.stderr
    assert compiles or "all row tiles or halves" in r.stderr


@pytest.mark.parametrize("phase,call,refusal", [
    ("GemmPhase<float, 1, 64, 64, 8>", "run(x, 72, 6, b, [&](int o0, int r, f32x4 (&acc)[1]) { x[o0 + r] = acc[0][0]; })", None),
    ("GemmPhase<float, 1, 64, 64, 8, 1, 1, true>", "run(x, 72, 6, b, [&](int o0, int r, f32x4 (&acc)[1]) { x[o0 + r] = acc[0][0]; })", "not swizzled"),
    ("GemmPhase<float, 1, 64, 64, 4>", "template run_before<4>(x, 72, 6, b, [&](int k, int o0, int r, f32x4 (&acc)[1]) { x[o0 + r + k] = acc[0][0]; }, []() {})", None),
    ("GemmPhase<float, 1, 64, 64, 4>", "template run_before<5>(x, 72, 6, b, [&](int k, int o0, int r, f32x4 (&acc)[1]) { x[o0 + r + k] = acc[0][0]; }, []() {})", "would never run"),
    ("GemmPhase<float, 1, 64, 64, 4>", "template run_rows<false, 4>(x, 72, 6, [&](int k, int r, f32x4 (&acc)[1]) { x[r + k] = acc[0][0]; })", None),
    ("GemmPhase<float, 1, 64, 64, 4>", "template run_rows<false, 5>(x, 72, 6, [&](int k, int r, f32x4 (&acc)[1]) { x[r + k] = acc[0][0]; })", "would never run")])
def test_phases_that_would_drop_or_misread_rows_do_not_compile(tmp_path, phase, call, refusal):
    """An epilogue has at most as many parts as the phase has k-fragments (four here), and run() does not read swizzled rows."""
    import subprocess
    from paper_2301_06051_amd import build
    if not os.path.exists(build.HIPCC):
        pytest.skip("no compiler")
    src = tmp_path / "phase.hip"
    src.write_text('#include "mma.h"\n'
                   "__global__ void k(const float* w, const float* b, float* x) {\n"
                   f"  {phase} phase(w, threadIdx.x >> 6);\n"
                   f"  phase.{call};\n"
                   "}\n")
    r = subprocess.run([build.HIPCC, *build.FLAGS, "--cuda-device-only", "-fsyntax-only", str(src)], capture_output=True, text=True)
    assert (r.returncode == 0) == (refusal is None), r.stderr
    assert refusal is None or refusal in r.stderr


def test_host_only_calls_work_without_a_gpu():
    """dsvt_partition_bound is pure host arithmetic: the set bound and a positive scratch size."""
    if not os.path.exists(LIB):
        pytest.skip("library not built")
    from paper_2301_06051_amd import binding as b
    cfg = b.part_cfg((468, 468, 1), (12, 12, 1), (6, 6, 0), 36, 1, 0)
    max_sets, max_tiles, ws = b.dsvt_partition_bound(cfg, 30000)
    assert max_sets == 30000 // 36 + 40 * 40 and ws > 0
    assert max_tiles == (30000 + 4 * max_sets) // 64 + 1 + 256
    with pytest.raises(b.DsvtError):
        b.dsvt_partition_bound(b.part_cfg((468, 468, 1), (12, 12, 1), (12, 0, 0), 36, 1, 0), 30000)
    with pytest.raises(b.DsvtError):
        b.dsvt_partition_bound(b.part_cfg((468, 468, 1), (12, 12, 1), (0, 0, 0), 36, 1, 6), 30000)      # inner orders are 0..5
    with pytest.raises(b.DsvtError):
        b.dsvt_partition_bound(b.part_cfg((468, 468, 32), (48, 48, 32), (0, 0, 0), 36, 1, 2), 30000)   # shuffled order: window volume <= 65536


def test_bench_refuses_more_than_one_gpu():
    """bench.py is single-GPU by design: any other --gpus value exits with a message before touching a device."""
    import subprocess
    import sys
    root = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
    r = subprocess.run([sys.executable, os.path.join(root, "bench.py"), "--gpus", "2"], capture_output=True, text=True, timeout=120)
    assert r.returncode == 2 and "single-GPU" in r.stderr and r.stdout.strip() == ""


def test_layer_kernels_of_long_frames_spill_nothing():
    """The layer's kernels for frames of several rounds of tiles: sets of up to 48 voxels, repeats masked or as keys, four shapes."""
    if not os.path.exists(LIB):
        pytest.skip("library not built")
    kernels = [k for k in _kernel_metadata(LIB) if "k_long_layer" in k[0]]
    assert len(kernels) == 8 and [k for k in kernels if k[1] or k[2] or k[3]] == []


def test_bench_reports_layer_traffic_only_for_the_sources_it_was_measured_with(tmp_path, monkeypatch):
    """bench.py takes the layer kernel's HBM bytes per launch from profiles/k_layer_hbm_traffic.txt, by workload, and
    only when the file's hash of layer.hip + mma.h is that of the sources in the tree."""
    import sys
    sys.path.insert(0, ROOT)
    import bench
    f = tmp_path / "traffic.txt"
    f.write_text("# comment\n"
                 f"workload=frame commit=abc1234 sources={bench.layer_source_hash()} fetch_kib=100 write_kib=28\n"
                 "workload=voxel commit=abc1234 sources=0000000000000000 fetch_kib=1 write_kib=1\n")
    monkeypatch.setattr(bench, "TRAFFIC_FILE", str(f))
    nbytes, where = bench.layer_traffic("frame")
    assert nbytes == 128 * 1024 and "abc1234" in where
    assert bench.layer_traffic("voxel")[0] is None and "other kernel sources" in bench.layer_traffic("voxel")[1]
    assert bench.layer_traffic("skewed") == (None, "not measured for this workload")
    monkeypatch.setattr(bench, "TRAFFIC_FILE", str(tmp_path / "missing.txt"))
    assert bench.layer_traffic("frame") == (None, "no traffic file")


def test_committed_traffic_file_matches_the_committed_kernel_sources():
    """The tracked traffic figures belong to the tracked layer.hip and mma.h (a change to either needs a new measurement)."""
    import sys
    sys.path.insert(0, ROOT)
    import bench
    for w in ("frame", "skewed", "voxel"):
        nbytes, where = bench.layer_traffic(w)
        assert nbytes is not None and nbytes > 0, (w, where)


def test_vfe_scratch_follows_the_way_of_counting():
    """A call whose few points do not pay for a counter per cell does not ask for the counters (grids of 1.5 M cells and 20
    more a point; 80,000 points; 8 M cells), and more points never ask for less."""
    if not os.path.exists(LIB):
        pytest.skip("library not built")
    from paper_2301_06051_amd import binding as b

    def size(grid, n, batch=1):
        cfg = b.VfeCfg(b.I32x3(*grid), batch, b.F32x3(-1.0, -1.0, -1.0), b.F32x3(0.5, 0.5, 0.5), 5, 5, b.DSVT_F32, None, None, 0)
        return b.dsvt_vfe_workspace_size(cfg, n, n)

    for grid, below, at in (((468, 468, 32), 79999, 80000), ((1500, 1000, 2), 74999, 75000), ((256, 256, 128), 79999, 80000)):
        counters = 4 * grid[0] * grid[1] * grid[2]
        assert size(grid, below) < counters <= size(grid, at)
        sizes = [size(grid, n) for n in (1, 500, 20000, below, at, at + 1, 400000)]
        assert sizes == sorted(sizes)
    assert size((468, 468, 8), 12500) < 4 * 468 * 468 * 8 <= size((468, 468, 8), 12610)
    assert size((256, 256, 129), 100000) < 4 * 256 * 256 * 129 and size((468, 468, 32), 100000, 2) < 4 * 2 * 468 * 468 * 32
    assert size((468, 468, 6), 1) >= 4 * 468 * 468 * 6


def test_bench_counts_the_pooling_operations_that_are_needed():
    """Two regions of one voxel, one of three, one of two: with masked holes those of one voxel need two products, else four."""
    import sys
    sys.path.insert(0, ROOT)
    import bench
    coords = [(0, 0, 0, 0), (0, 0, 0, 4), (0, 0, 0, 5), (0, 0, 0, 7), (1, 0, 0, 4), (0, 1, 0, 1), (0, 1, 0, 2)]
    assert bench.pool_flops(coords, (1, 1, 4), 10, 0) == 200 * (2 * 7 + 2 * 4)
    assert bench.pool_flops(coords, (1, 1, 4), 10, 1) == 200 * (2 * 5 + 2 * 2 + 2 * 2)
