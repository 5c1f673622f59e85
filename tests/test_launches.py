"""What the library launches, recorded without a GPU (launch_recorder.c stands in for the HIP
runtime): routes, grids and buffers of layers that are too large or too odd to run in a test."""
import os
import re
import shutil
import subprocess

import pytest

import paper_2101_03961_amd as sw

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
pytestmark = pytest.mark.skipif(shutil.which("gcc") is None, reason="needs gcc")


@pytest.fixture(scope="module")
def recorder(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("launches") / "launch_recorder")
    subprocess.run(["gcc", "-O1", "-Wall", "-Werror", "-rdynamic", "-I", os.path.join(ROOT, "include"), "-o", exe,
                    os.path.join(ROOT, "tests", "launch_recorder.c"), "-ldl"], check=True)

    def record(*calls):
        """[(status, workspace address, bytes, [(kernel, grid, block, lds, args)])] of the calls."""
        lines = "".join(" ".join(str(v) for v in c) + "\n" for c in calls)
        run = subprocess.run([exe, sw.library_path()], input=lines, capture_output=True, text=True, check=True)
        out, launches = [], []
        for line in run.stdout.splitlines():
            word = line.split()
            if word[0] == "launch":
                v = [int(t) for t in word[2:]]
                launches.append((word[1], tuple(v[:3]), tuple(v[3:6]), v[6], v[7:]))
            elif word[0] == "call":
                out.append((int(word[1]), int(word[2]), int(word[3]), launches))
                launches = []
        assert len(out) == len(calls)
        return out
    return record


def call(what, T, d, f, E, cf, dtype="bf16", ffn="relu", n=1, dropout=0.0, jitter=0.0, ntlb=0, fused=False, bias=False):
    return (what, T, d, f, E, cf, 1 if dtype == "bf16" else 0, 1 if ffn == "geglu" else 0, n, dropout, jitter, ntlb,
            int(fused), int(bias))


# The router's weights are split for the forward pass and, where its backward pass reads them, for that:
# the second buffer is written only if it is there, and lies inside the workspace then.
@pytest.mark.parametrize("kw,backward_reads", [
    (dict(T=262144, d=768, f=3072, E=2048, cf=1.0, ffn="geglu"), False),   # more logits than a descriptor spans
    (dict(T=524288, d=512, f=1536, E=1024, cf=1.0, ffn="geglu"), False),
    (dict(T=1 << 22, d=64, f=64, E=128, cf=1.0, jitter=0.01), False),
    (dict(T=8192, d=768, f=3072, E=2048, cf=1.0, ffn="geglu"), True),
    (dict(T=32768, d=768, f=3072, E=128, cf=1.0, jitter=0.01), False),     # the one-kernel backward reads W_r
])
def test_split_router_weights_stay_in_the_workspace(recorder, kw, backward_reads):
    (status, base, size, launches), = recorder(call("forward", **kw))
    assert status == 0
    (_, _, _, _, (_, wsplit, wsplit_b)), = [k for k in launches if "router_split_kernel" in k[0]]
    assert base <= wsplit < base + size
    assert (wsplit_b != 0) == backward_reads
    if wsplit_b:
        tiles = -(-kw["E"] // 128)
        assert base <= wsplit_b and wsplit_b + tiles * kw["d"] * 512 <= base + size


# Prefix sums of the block histograms: by the assign kernel itself with few experts, groups and token blocks
# (it sums all of them in every block), by the scan kernel otherwise.
@pytest.mark.parametrize("T,E,n,fused,scan", [
    (64, 128, 1, False, False), (8192, 256, 1, False, False), (8193, 256, 1, False, True),
    (64, 260, 1, False, True), (32768, 4096, 1, False, True), (64, 4096, 1, False, True),
    (8192, 128, 2, False, False), (4096, 128, 4, False, False), (8192, 128, 4, False, True),
    (2048, 64, 8, False, True), (64, 128, 1, True, True)])
def test_scan_kernel_beside_many_experts_groups_or_blocks(recorder, T, E, n, fused, scan):
    (status, _, _, launches), = recorder(call("forward", T, 64, 64, E, 1.25 * max(1.0, n * E / T), n=n, fused=fused))
    assert status == 0
    assert any("route_scan_kernel" in k[0] for k in launches) == scan
    assert sum("assign_kernelILb%d" % (not scan) in k[0] for k in launches) == 1


# Tile of the products whose rows are tokens, by rows per expert (the first four template arguments of the
# kernel: 32-column tiles per wave, waves, 32-row tiles per wave, waves): no tall tile for a handful of rows.
@pytest.mark.parametrize("T,d,f,E,cf,first,second", [
    (240, 184, 664, 232, 1.0, "1,4,1,1", "1,4,1,1"), (2048, 264, 2704, 256, 1.0, "1,4,1,1", "1,4,1,1"),
    (503, 264, 2000, 308, 1.0, "1,4,1,1", "1,4,1,1"), (64, 768, 3072, 128, 8.0, "1,4,1,1", "1,4,1,1"),
    (4096, 768, 3072, 128, 1.25, "2,4,2,1", "2,4,2,1"), (8192, 768, 3072, 128, 1.25, "3,4,4,2", "3,4,4,2"),
    (65536, 768, 3072, 128, 1.0, "3,4,4,2", "3,4,4,2"), (16384, 4096, 10240, 64, 1.25, "2,4,5,2", "2,4,5,2"),
    # (experts of 64 row tiles and more, one column tile: cut into pieces if there are no more than 64)
    (65536, 136, 264, 8, 1.96875, "3,4,4,2", "2,4,4,2"), (65536, 136, 264, 8, 2.0, "3,4,4,2", "2,4,4,2"),
    (65536, 200, 264, 8, 2.0, "3,4,4,2", "2,4,4,2"), (65536, 136, 264, 4, 2.0, "3,4,4,2", "2,4,4,2"),
])
def test_tile_follows_the_rows_of_an_expert(recorder, T, d, f, E, cf, first, second):
    (status, _, _, launches), = recorder(call("forward", T, d, f, E, cf))
    assert status == 0
    tiles = [",".join(re.findall(r"Li(\d+)E", k[0])[:4]) for k in launches if "gemm_rows_kernel" in k[0]]
    assert tiles == [first, second]


# Kernel of the weight gradients (first layer, second layer) by size: persistent blocks with the long side along
# the smaller dimension unless that pads more, smaller tiles for few experts, 256 x 256 where that fills the rounds.
@pytest.mark.parametrize("T,d,f,E,cf,first,second", [
    (65536, 768, 3072, 128, 1.0, "wgrad 4,2,3,4", "wgrad 3,4,4,2"),
    (16384, 4096, 10240, 64, 1.25, "wgrad 4,2,3,4", "wgrad 3,4,4,2"),
    (65536, 1024, 2816, 128, 1.25, "wgrad 3,4,4,2", "wgrad 4,2,3,4"),   # the other way: 32 tiles instead of 33
    (2400, 264, 904, 120, 1.25, "wgrad 4,2,3,4", "wgrad 3,4,4,2"),
    (9000, 264, 760, 80, 1.25, "wgrad 4,2,3,4", "wgrad 3,4,4,2"),
    (2400, 264, 904, 120, 4.0, "wgrad 4,2,3,4", "wgrad 3,4,4,2"),
    (2500, 264, 904, 250, 4.0, "wgrad 4,2,3,4", "wgrad 3,4,4,2"),
    (9000, 264, 760, 80, 0.007, "rows 2,2,4,2", "rows 2,2,4,2"),        # no slots
    (32768, 512, 1024, 32, 1.0, "bf16", "bf16"),
    (512, 768, 3072, 128, 4.0, "rows 2,2,4,2", "rows 2,2,4,2"),
    # rows that share lines, more than 512 MB: guarded stores, up to 32 tokens per expert if column tiles are neighbours
    (500, 1080, 2408, 100, 4.0, "rows 2,2,4,2 guarded", "rows 2,2,4,2 guarded"),
    (2400, 1080, 2408, 100, 1.25, "wgrad 4,2,3,4", "rows 2,2,4,2 guarded"),
    (3200, 1080, 2408, 100, 1.25, "wgrad 4,2,3,4", "wgrad 3,4,4,2"),
    (384, 3000, 6008, 32, 1.25, "wgrad 4,2,3,4", "wgrad 3,4,4,2"),
    (490, 1080, 2408, 98, 4.0, "rows 2,2,4,2", "rows 2,2,4,2"),         # less than 512 MB
    (500, 1088, 2432, 100, 4.0, "rows 2,2,4,2", "rows 2,2,4,2"),        # whole lines
])
def test_kernel_of_the_weight_gradients(recorder, T, d, f, E, cf, first, second):
    (status, _, _, launches), = recorder(call("backward", T, d, f, E, cf))
    assert status == 0
    got = []
    for name, *_ in launches:
        m = re.search(r"gemm_(rows|wgrad|bf16)_kernelI((?:L[ib]\d+E)*)", name)
        flags = re.findall(r"Lb([01])E", m[2]) if m else []
        if m and (m[1] == "wgrad" or m[1] == "rows" and flags[-2] == "1" or m[1] == "bf16" and flags[:2] == ["1", "1"]):
            got.append(m[1] + ("" if m[1] == "bf16" else " " + ",".join(re.findall(r"Li(\d+)E", m[2])[:4])) +
                       (" guarded" if m[1] == "rows" and flags[-1] == "1" else ""))
    assert got[:2] == [first, second]


# Small layers: the first layer's data gradient and both weight gradients in one launch (tiles of four waves and
# weights that fit the memory-side cache), else one launch each.
@pytest.mark.parametrize("T,d,f,E,cf,data,weights", [
    (5003, 392, 1000, 10, 1.25, "1,4,3,1,2", "2,2,2,2,2"), (60000, 128, 512, 16, 1.0, "1,4,3,1,2", "2,2,2,2,2"),
    (4096, 256, 1024, 64, 1.0, "1,4,3,1,2", "2,2,4,2,1"), (300, 512, 2048, 16, 2.0, "1,4,1,1,3", "2,2,4,2,1"),
    (512, 768, 3072, 128, 4.0, None, None), (65536, 768, 3072, 128, 1.0, None, None),
])
def test_small_layers_take_three_products_in_one_launch(recorder, T, d, f, E, cf, data, weights):
    (status, _, _, launches), = recorder(call("backward", T, d, f, E, cf))
    assert status == 0
    got = [re.findall(r"Li(\d+)E", k[0]) for k in launches if "gemm_rows_backward" in k[0]]
    assert [(",".join(g[:5]), ",".join(g[5:])) for g in got] == ([(data, weights)] if data else [])
    # the masked gradient, and the three others once
    assert sum("gemm_rows" in k[0] or "gemm_wgrad" in k[0] for k in launches) == (2 if data else 4)


# Input jitter on bf16 tokens: in the one-kernel router, or planes of x * m for large layers of many experts.
@pytest.mark.parametrize("T,d,E,planes", [
    (16384, 128, 128, False), (16385, 128, 128, True), (10000, 768, 128, False), (10200, 768, 128, True), (65536, 768, 64, False),
    (65536, 768, 68, True), (65536, 768, 127, False), (2280, 512, 256, False), (2300, 512, 256, True), (64, 1024, 132, False),
    (64, 1032, 132, True), (64, 1032, 128, False), (512, 64, 260, True)])
@pytest.mark.parametrize("fused", [False, True])
def test_route_of_input_jitter(recorder, T, d, E, planes, fused):
    (status, _, _, launches), = recorder(call("forward", T, d, 512, E, 4.0, jitter=0.01, fused=fused))
    assert status == 0
    assert any("jitter_split" in k[0] for k in launches) == planes
    assert any("router_block_kernel" in k[0] for k in launches) != planes


# The router's weight gradient: its parts beside the experts' where those are small, or fp32 ("beside"), which saves a launch
# for the parts and one for their sums; in a launch of their own ("parts"); on the matrix cores, or the vector ALUs.  Whether a
# layer fits the static scratch, whose calls have no backward pass, only moves the parts (1050 x 512 x 2600).
@pytest.mark.parametrize("T,d,f,E,cf,kw,form", [
    (5003, 392, 1000, 10, 1.25, dict(bias=True), "beside"), (256, 64, 256, 4, 1.25, dict(dtype="f32"), "beside"),
    (8192, 768, 3072, 32, 1.25, dict(dtype="f32", bias=True), "beside"), (1050, 512, 2048, 16, 2.0, dict(), "beside"),
    (1050, 512, 2048, 16, 2.0, dict(jitter=0.01), "beside"), (1050, 512, 2600, 16, 2.0, dict(), "parts"),
    (1050, 512, 2600, 16, 2.0, dict(jitter=0.01), "parts"), (1050, 512, 2720, 16, 2.0, dict(), "parts"),
    (512, 512, 3072, 128, 1.25, dict(), "parts"), (736, 1536, 112, 92, 1.25, dict(), "mfma"),
    (1513, 1312, 48, 16, 2.0, dict(jitter=0.01), "vector"),   # room for a quarter of the parts
    (8192, 768, 3072, 128, 1.25, dict(), "mfma"), (500, 64, 256, 300, 4.0, dict(dtype="f32"), "vector"),
    (5003, 392, 1000, 10, 1.25, dict(fused=True), "vector"), (2000, 512, 2048, 16, 1.25, dict(fused=True), "mfma"),
    (2000, 512, 2048, 16, 1.25, dict(fused=True, jitter=0.01), "parts"),
    (4096, 768, 3072, 128, 1.25, dict(fused=True, jitter=0.01, bias=True), "parts"),
    (65536, 768, 3072, 128, 1.25, dict(fused=True, jitter=0.01), "mfma"),
    # near the static scratch's limit, but beyond it without parts too: nothing moves
    (7900, 296, 208, 64, 1.0, dict(n=4, dropout=0.1), "beside"), (2470, 768, 48, 64, 1.0, dict(dtype="f32"), "beside"),
    # many tokens to many experts: on the matrix cores where those take its operands
    (8192, 256, 64, 64, 1.25, dict(), "beside"), (8193, 256, 64, 64, 1.25, dict(), "mfma"), (8193, 256, 64, 32, 1.25, dict(), "beside"),
    (8193, 256, 64, 62, 1.25, dict(), "beside"), (4096, 384, 64, 96, 1.25, dict(), "mfma"),
    (4096, 512, 8192, 16, 1.25, dict(), "parts"), (4100, 512, 8192, 16, 1.25, dict(), "mfma"),
    # memory for few parts: of many experts, from 1e9 products on
    (6050, 5000, 64, 33, 1.25, dict(), "parts"), (6072, 5000, 64, 33, 1.25, dict(), "vector"),
    (2850, 5000, 64, 70, 1.25, dict(dtype="f32"), "beside"), (2870, 5000, 64, 70, 1.25, dict(dtype="f32"), "vector"),
    (6072, 5000, 64, 64, 1.25, dict(dtype="f32"), "beside"), (12000, 5000, 64, 30, 1.25, dict(), "parts"),
    (20000, 768, 64, 140, 1.25, dict(dtype="f32"), "vector"), (20000, 768, 64, 133, 1.25, dict(), "parts"),
])
def test_router_weight_gradient_beside_the_experts(recorder, T, d, f, E, cf, kw, form):
    (status, base, size, launches), = recorder(call("backward", T, d, f, E, cf, **kw))
    assert status == 0
    kernels = {"parts": "router_wgrad_kernel", "mfma": "router_dWr_mfma_kernel", "vector": "router_dWr_kernel"}
    got = [k for k, name in kernels.items() if any(name in launch[0] for launch in launches)]
    assert got == ([] if form == "beside" else [form])
    assert any("reduce" in k[0] for k in launches) == (form in ("mfma", "vector"))


# How many parts it comes in, in tiles of 4096 elements: one per 32 tokens up to 64, one per 128 while the blocks run at a time
# (512), one per 512; up to 256, and 16 MB; each a multiple of 32 tokens.
@pytest.mark.parametrize("T,d,E,parts", [(1, 512, 30, 1), (33, 512, 30, 2), (2048, 512, 30, 64), (12000, 512, 30, 75),
                                         (40000, 512, 30, 125), (100000, 512, 30, 241), (200000, 512, 30, 250), (40000, 4096, 30, 34)])
def test_parts_of_the_router_weight_gradient(recorder, T, d, E, parts):
    (status, _, _, launches), = recorder(call("backward", T, d, 8192, E, max(1.25, 4 * E / T)))
    assert status == 0
    (grid,) = [k[1] for k in launches if "router_wgrad_kernel" in k[0]]
    assert grid == (-(-d // 128) * parts, 1, 1)


# The sums over its parts: blocks of the launch that computes dx, each once (256 sums each, and db_r's), behind those of 128
# tokens by a range of columns.
@pytest.mark.parametrize("T,d,f,E,cf,kw,dx_blocks", [
    (64, 4096, 256, 128, 4.0, dict(), 64), (300, 4096, 1024, 98, 4.0, dict(bias=True), 3 * 64),
    (1000, 2048, 256, 256, 2.0, dict(dtype="f32", bias=True), 8 * 64), (256, 64, 256, 4, 1.25, dict(dtype="f32"), 2),
    (60000, 128, 512, 16, 1.0, dict(bias=True), 469 * 2),
])
def test_sums_of_the_router_weight_gradient_are_launched_once(recorder, T, d, f, E, cf, kw, dx_blocks):
    (status, _, _, launches), = recorder(call("backward", T, d, f, E, cf, **kw))
    assert status == 0
    (grid,) = [k[1] for k in launches if "router_dx" in k[0]]
    assert grid == (dx_blocks + -(-d * E // 256) + (-(-E // 32) if kw.get("bias") else 0), 1, 1)


# The combine: in the second GEMM's epilogue (small tiles, fp32), which saves a launch unless re-routing stages follow the
# assignment of the slots; else a pass of its own.
@pytest.mark.parametrize("T,d,f,E,cf,dtype,rounds,own", [
    (45, 80, 176, 29, 2.6, "bf16", 0, False), (45, 80, 176, 29, 2.6, "bf16", 1, True),
    (256, 64, 256, 4, 1.25, "f32", 0, False), (256, 64, 256, 4, 1.25, "f32", 3, True),
    (65536, 768, 3072, 128, 1.0, "bf16", 0, True),
])
def test_combine_in_the_epilogue_or_as_a_pass(recorder, T, d, f, E, cf, dtype, rounds, own):
    (status, _, _, launches), = recorder(call("forward", T, d, f, E, cf, dtype=dtype, ntlb=rounds))
    assert status == 0
    assert sum("combine_kernel" in k[0] for k in launches) == (1 if own else 0)
    assert not any("zero_dropped" in k[0] for k in launches)


# fp32 products: matrix cores while an expert's matrices fit a buffer descriptor, else the FMA kernel
@pytest.mark.parametrize("T,d,f,E,cf,kernel", [(256, 64, 256, 4, 1.25, "gemm_f32_mfma_kernel"),
                                               (101, 12, 516, 2, 20800.0, "gemm_f32_kernel"),
                                               (8, 4096, 131072, 1, 1.0, "gemm_f32_kernel")])
def test_fp32_products_by_size(recorder, T, d, f, E, cf, kernel):
    for what, n in (("forward", 2), ("backward", 4)):
        (status, _, _, launches), = recorder(call(what, T, d, f, E, cf, dtype="f32"))
        assert status == 0
        assert [kernel in k[0] for k in launches if "gemm_f32" in k[0]] == [True] * n


# Passes with one wave per token, beyond 2^26 tokens: the same limit
@pytest.mark.parametrize("kw", [dict(), dict(fused=True), dict(ntlb=2), dict(fused=True, ntlb=1), dict(dtype="f32", jitter=0.1)])
def test_grids_of_very_many_tokens(recorder, kw):
    T = (1 << 26) + 12
    for what in ("forward", "backward"):
        (status, _, _, launches), = recorder(call(what, T, 8, 8, 4, 1.0, bias=True, **kw))
        assert status == 0
        for name, grid, block, _, _ in launches:
            assert all(g * b < 1 << 32 for g, b in zip(grid, block)) and grid[1] <= 65536, name
            if "combine" in name or "dispatch_kernel" in name or "dropped" in name or "gate_grad" in name:
                assert grid[0] * grid[1] * 4 >= T, name


# Layers whose expert GEMMs have more tiles than one grid dimension takes (2^32 threads): many experts of
# extreme widths.  Every launch stays inside the limit, and the tiles are all there.
@pytest.mark.parametrize("what", ["forward", "backward"])
@pytest.mark.parametrize("dtype,d,f,cf", [("bf16", 8, 1 << 20, 1.0), ("bf16", 8, (1 << 19) + 136, 1.0), ("f32", 4, 1 << 20, 1.0)])
def test_grids_stay_inside_the_launch_limits(recorder, what, dtype, d, f, cf):
    E = 4096
    (status, _, _, launches), = recorder(call(what, E, d, f, E, cf, dtype=dtype))
    assert status == 0
    for name, grid, block, lds, _ in launches:
        assert all(g * b < 1 << 32 and g > 0 for g, b in zip(grid, block)), name
        assert max(grid[1:]) <= 65536 and lds <= 160 * 1024, name
    # the first one: f columns of one row tile per expert
    name, grid = [k[:2] for k in launches if "gemm_" in k[0]][0]
    ip, wp = (int(v) for v in re.findall(r"Li(\d+)E", name)[:2]) if dtype == "bf16" else (1, 2)   # FMA kernel: 64 columns
    assert grid[0] * grid[1] * grid[2] >= E * -(-f // (32 * ip * wp))


# Weight gradients of a 256 x 128 tile: three blocks per CU where an expert has more than one step of 64 slots, else two
# (sixth argument of the kernel's template).
@pytest.mark.parametrize("T,d,f,E,blocks", [(39584, 752, 2696, 8, 3), (512, 768, 1536, 128, 2), (512, 1080, 2408, 208, 2)])
def test_blocks_per_cu_of_the_tall_weight_gradient_tile(recorder, T, d, f, E, blocks):
    (status, _, _, launches), = recorder(call("backward", T, d, f, E, 1.25))
    assert status == 0
    tall = [k[0] for k in launches if "gemm_rows_kernelILi2ELi2ELi4ELi2ELi1E" in k[0]]
    assert tall and all("Li1ELi%dELb1E" % blocks in k for k in tall)
