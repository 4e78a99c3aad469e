"""Where the launches of a product put their partial tiles, over the sizes, layouts and alignments that the entry points
take.  Runs on the CPU: launch_plans.cpp stands in for the HIP runtime and looks at the arguments."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
PKG = os.path.join(ROOT, "paper_2508_04355_amd")


@pytest.fixture(scope="module")
def plans(tmp_path_factory):
    if not os.path.exists(os.path.join(PKG, "libgecc.so")):
        from paper_2508_04355_amd import build
        build.build(verbose=False)
    rocm = os.environ.get("ROCM_PATH", "/opt/rocm")
    exe = str(tmp_path_factory.mktemp("plans") / "launch_plans")
    subprocess.run(["g++", "-O1", "-std=c++17", "-D__HIP_PLATFORM_AMD__", "-I" + os.path.join(ROOT, "include"), "-I" + os.path.join(PKG, "csrc"),
                    "-I" + os.path.join(rocm, "include"), os.path.join(ROOT, "tests", "launch_plans.cpp"), "-o", exe, "-rdynamic",
                    "-L" + PKG, "-l:libgecc.so", "-Wl,-rpath," + PKG, "-L" + os.path.join(rocm, "lib"), "-lamdhip64",
                    "-Wl,-rpath," + os.path.join(rocm, "lib")], check=True)
    return exe


def routes(exe, calls, what="routes"):
    """[(result, [kernel names])] of calls (entry, n, k, m, batch, dtype, trans_a, trans_b); what = "grids": a name is followed by ":" and
    its workgroups."""
    r = subprocess.run([exe, what], input="\n".join(" ".join(str(x) for x in c) for c in calls), capture_output=True, text=True, timeout=120)
    lines = [x.split() for x in r.stdout.splitlines() if not x.startswith("BAD")]
    assert r.returncode == 0 and len(lines) == len(calls), r.stdout + r.stderr
    return [(int(x[0]), x[1:]) for x in lines]


def test_partial_tiles_stay_in_their_part_of_the_workspace(plans):
    """Every k-split launch of gemm_tile (also where the kernel with 256 x 256 tiles was planned and refuses the operands)
    writes no more than the workspace has for it."""
    r = subprocess.run([plans], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stdout + r.stderr


@pytest.mark.parametrize("ta,tb", [(0, 0), (0, 1), (1, 0), (1, 1)])
def test_products_that_go_in_fp32_tiles_of_128_by_256(plans, ta, tb):
    """The sizes that tests of that kernel use reach it (and the others, to which it is compared, do not)."""
    from test_tiles_and_scans import HALVES_OTHER_BATCH, HALVES_SHAPES, SMALL_CASES, WIDE_CASES
    for cases, kernel in ((WIDE_CASES, "gemm_f32_wide"), (SMALL_CASES, "gemm_tileILi0ELb%dELb%dELi64E" % (not ta, tb))):
        for entry in ("plain", "multiply"):
            for _, names in routes(plans, [(entry,) + shape + (batch, 0, ta, tb) for shape, batch in cases]):
                assert kernel in names[-1] and sum("gemm" in x for x in names) == 1, names
    for n, k, m in HALVES_SHAPES:
        (_, wide), (_, other) = routes(plans, [("plain", n, k, m, 256, 0, ta, tb), ("plain", n, k, m, HALVES_OTHER_BATCH, 0, ta, tb)])
        assert len(wide) == 1 and "gemm_f32_wide" in wide[0]
        assert len(other) == 1 and "gemm_tile" in other[0] and "ELi128E" in other[0]


def test_sums_of_32_chunks_are_left_to_their_readers_and_of_33_are_not(plans):
    """Both sides of that limit, at sizes of test_sums_left_to_their_readers: the parity blocks ride in the product's launch
    in either case, the encodings share a launch where A_P's chunks stay as they are."""
    (_, left), (_, done) = routes(plans, [("protected", n, 72, 130, 1, 0, 0, 0) for n in (4096, 4097)])
    assert any("scan_pair" in x for x in left) and not any("scan_pair" in x for x in done)
    assert len(done) == len(left) + 1 and not any("rowdot" in x or "coldot" in x for x in left)


@pytest.mark.parametrize("dtype", [0, 1])
def test_two_parity_blocks_go_in_the_kernel_of_their_kind(plans, dtype):
    """Column scans (TN) in the one for column scans, row scans (NT) in the one for rows; many short rows in the one with
    a wavefront for eight of them."""
    tn, nt, short = [names for _, names in routes(plans, [("protected", 2048, 2048, 2048, 1, dtype, 1, 0), ("protected", 2048, 2048, 2048, 1, dtype, 0, 1),
                                                          ("protected", 512, 128, 512, 256, dtype, 0, 1)])]
    for names, kind in ((tn, 2), (nt, 0), (short, 1)):
        assert sum("scan_pairILi%dELb0ELi%dE" % (dtype, kind) in x for x in names) == 1, names


@pytest.mark.parametrize("dtype,shape,batch,one_pass",
                         [(0, (512, 512, 512), 64, True), (0, (512, 512, 512), 63, False), (0, (512, 252, 512), 260, False),
                          (0, (512, 252, 512), 261, True), (1, (512, 512, 512), 127, False), (1, (512, 512, 512), 128, True)])
def test_operands_that_the_one_pass_scan_takes(plans, dtype, shape, batch, one_pass):
    """64 MiB, and 2^25 elements where the rows are shorter than 256."""
    n, k, m = shape
    (_, names), = routes(plans, [("protected", n, k, m, batch, dtype, 0, 1)])
    assert any("tile_scan" in x for x in names) == one_pass, names


def test_calls_of_many_workgroups_are_taken(plans):
    """Launches of which each fits what one may have (2^32 threads) are not put into one that does not: scans of many batch
    items, fp32 tiles of twice the threads."""
    calls = [("protected", 7, 4128, 7, 65535, 1, ta, tb) for ta in (0, 1) for tb in (0, 1)]
    calls += [("protected", 23, 9514, 1, 52984, 1, 1, 0), ("protected", 11307, 9, 5, 65535, 1, 0, 1), ("protected", 4, 2, 10111, 65535, 1, 0, 1),
              ("protected", 6, 8000, 7, 65535, 0, 1, 1)]
    calls += [("plain", 128, 256, 1664, 1 << 20, 0, 0, 0), ("plain", 128, 256, 1664, 1290000, 0, 0, 1)]     # 7.3 and 9.0 million tiles of 128 x 256
    r = routes(plans, calls)
    assert [rc for rc, _ in r] == [0] * len(calls)
    # two scans of one kind go in two launches only there
    few = routes(plans, [("protected", 7, 4128, 7, 60, 1, 1, 0)])[0][1]
    encodings = "scan_pairILi1ELb1E"      # (index weights)
    assert any(encodings in x for x in few) and not any(encodings in x for x in r[2][1])
    assert "gemm_f32_wide" in r[-2][1][0] and "gemm_tile" in r[-1][1][0]


@pytest.mark.parametrize("ta,tb", [(0, 0), (0, 1), (1, 0), (1, 1)])
def test_bf16_products_either_kernel_takes(plans, ta, tb):
    """Which one they go to, by size and layout: gemm_tile with the parity scans in its launch where that saves launches (a protected
    product), the faster kernel for a product on its own."""
    def product(entry, n, k, m):
        rc, names = routes(plans, [(entry, n, k, m, 1, 1, ta, tb)])[0]
        assert rc == 0
        return [x for x in names if "gemm" in x][0], sum("dot" in x or "scan" in x for x in names)
    two_launches = ta == tb
    for n, k, m in ((2048, 2048, 2048), (2560, 2560, 2560), (3072, 1024, 3072), (4096, 512, 2048)):
        name, scans = product("protected", n, k, m)
        assert ("gemm_tile" in name) == two_launches and (scans <= 3 if two_launches else scans >= 2)
        assert "gemm_bf16_256" in product("plain", n, k, m)[0]
    for n, k, m in ((256, 256, 256), (1280, 7296, 2304), (1024, 4096, 4096)):
        assert "gemm_tile" in product("protected", n, k, m)[0] and "gemm_tile" in product("plain", n, k, m)[0]
    for n, k, m in ((4096, 4096, 4096), (3072, 3072, 3072)):
        assert "gemm_bf16_256" in product("protected", n, k, m)[0]


@pytest.mark.parametrize("ta,tb", [(0, 0), (0, 1), (1, 0), (1, 1)])
def test_bf16_products_of_ragged_sizes_go_by_the_same_rule(plans, ta, tb):
    """Aligned sizes that are no multiples of a tile."""
    for n, k, m in ((2000, 1024, 2000), (2000, 512, 2000), (3000, 512, 3000), (2056, 2048, 2056), (1000, 512, 776), (520, 256, 264), (4040, 4032, 4008)):
        (rc, names), = routes(plans, [("protected", n, k, m, 1, 1, ta, tb)])
        assert rc == 0
        scans = [x for x in names if "dot" in x or "scan" in x]
        tile = bool(_has(names, "gemm_tile"))
        assert tile != bool(_has(names, "gemm_bf16_256")) and tile == ((n, k, m) == (520, 256, 264) or (n < 4000 and ta == tb)), names
        assert len(scans) <= 3 if tile else len(scans) >= 2, names


@pytest.mark.parametrize("ta,tb", [(0, 0), (0, 1), (1, 0), (1, 1)])
def test_products_on_their_own_go_to_the_faster_kernel(plans, ta, tb):
    """Also where a protected product would have tiles of 64 (4096 x 192 x 4096: 18.4 us in 256 x 256 tiles, 23.0 in tiles of 64)."""
    from test_tiles_and_scans import ALONE_SHAPE
    for (n, k, m), kernel in (((4096, 192, 4096), "gemm_bf16_256"), ((3072, 128, 4096), "gemm_bf16_256"), ((2048, 1024, 2048), "gemm_bf16_256"),
                              (ALONE_SHAPE, "gemm_bf16_256"), ((1024, 1024, 1024), "gemm_tile"), ((1536, 4224, 768), "gemm_tile")):
        (rc, names), = routes(plans, [("plain", n, k, m, 1, 1, ta, tb)])
        assert rc == 0 and len(names) == 1 + ("zero_words" in names[0]) and kernel in names[-1], names
    if not ta and not tb:
        (_, names), = routes(plans, [("protected",) + ALONE_SHAPE + (1, 1, ta, tb)])
        assert any("gemm_tileILi1E" in x and "ELi64E" in x for x in names), names


@pytest.mark.parametrize("ta,tb", [(0, 0), (0, 1), (1, 0), (1, 1)])
def test_products_whose_scans_do_not_ride_go_to_the_faster_kernel(plans, ta, tb):
    """More than 2048 tiles of 64: the parity scans have launches of their own beside either kernel, and nothing is saved by the slower one."""
    for n, k, m in ((4096, 192, 4096), (3072, 128, 4096)):
        (rc, names), = routes(plans, [("protected", n, k, m, 1, 1, ta, tb)])
        assert rc == 0 and any("gemm_bf16_256" in x for x in names), names


@pytest.mark.parametrize("ta,tb", [(0, 0), (0, 1), (1, 0), (1, 1)])
def test_batches_whose_scans_do_not_ride_go_to_the_faster_kernel(plans, ta, tb):
    """Items of 128 columns fill half of a 256 x 256 tile (128 x 1280 x 512 x 100 NN: 85 us in tiles of 128, 104 in those)."""
    for n, k, m, batch in ((128, 1280, 512, 100), (128, 1664, 1024, 54), (1088, 1792, 128, 41), (4608, 1536, 128, 12)):
        (rc, names), = routes(plans, [("protected", n, k, m, batch, 1, ta, tb)])
        assert rc == 0 and _has(names, "gemm_tileILi1E") and not _has(names, "gemm_bf16_256"), names


@pytest.mark.parametrize("shape,batch,per_item", [((4096, 4096, 4096), 1, 16), ((512, 512, 512), 256, 1), ((512, 512, 512), 128, 2), ((1024, 256, 1024), 200, 1),
                                                  ((2047, 24, 100), 130, 1), ((2048, 24, 100), 130, 3), ((100, 24, 4096), 256, 2), ((4096, 24, 100), 257, 1),
                                                  ((16384, 32, 512), 60, 4), ((2048, 64, 512), 128, 2), ((2048, 64, 512), 129, 3), ((16384, 32, 512), 1, 64)])
def test_workgroups_of_a_repair(plans, shape, batch, per_item):
    """One for 256 lines of an item, at most 256 in all or, of more than 128 items of lines of 2048 and longer, 512."""
    for dtype in (0, 1):
        (rc, names), = routes(plans, [("correct",) + shape + (batch, dtype, 0, 0)], "grids")
        assert rc == 0 and [x.split(":")[1] for x in names if "repair_kernel" in x] == [str(per_item * batch)], names


def _has(names, what):
    return [x for x in names if what in x]


@pytest.mark.parametrize("dtype", [0, 1])
def test_column_scans_in_vectors_of_either_width(plans, dtype):
    """The sizes that tests of them use: index weights and explicit ones, in a launch of their own and two in one."""
    from test_tiles_and_scans import WIDE_SCANS
    (n, k, m), batch = WIDE_SCANS
    for shape, b, half in (((n, k, m), batch, 0), ((129, 130, 131), 1, 1), ((260, 300, 16200), 1, 1)):
        nn, nt, tn = [names for _, names in routes(plans, [("protected",) + shape + (b, dtype) + t for t in ((0, 0), (0, 1), (1, 0))])]
        if not half:          # (elsewhere the parity scans ride, or the two encodings share a launch)
            for idxw in (1, 0):
                assert _has(nn, "coldot_stage1ILi%dELb%dELb0ELb0ELb0E" % (dtype, idxw)), nn
            assert _has(tn, "scan_pairILi%dELb0ELi2ELb0E" % dtype), tn
        assert _has(nt, "scan_pairILi%dELb1ELi0ELb%dE" % (dtype, half)) or _has(nt, "scan_pairILi%dELb1ELi1ELb%dE" % (dtype, half)), nt
        staged = routes(plans, [("encode_a",) + shape + (b, dtype, 0, 0)])[0][1]
        assert _has(staged, "coldot_stage1ILi%dELb1ELb0E" % dtype) and _has(staged, "ELb%dEEEv" % half), staged


@pytest.mark.parametrize("ta,tb", [(0, 0), (0, 1), (1, 0), (1, 1)])
def test_bf16_products_that_carry_their_scans(plans, ta, tb):
    """The sizes that a test of them uses: tiles and ranges (by the workgroups of the product alone), no scan behind the encodings."""
    from test_tiles_and_scans import BESIDE_CASES
    for (n, k, m), tile, ranges in BESIDE_CASES:
        (_, plain), (_, multiply) = routes(plans, [(e, n, k, m, 1, 1, ta, tb) for e in ("plain", "multiply")], "grids")
        assert not _has(multiply, "dot") and not _has(multiply, "scan") and len(_has(multiply, "gemm_tileILi1E")) == 1, multiply
        name, grid = plain[-1].split(":")
        assert "gemm_tileILi1E" in name and "ELi%dEEEv" % tile in name and int(grid) == -(-n // tile) * -(-m // tile) * ranges, plain


@pytest.mark.parametrize("ta,tb", [(0, 0), (0, 1), (1, 0), (1, 1)])
def test_bf16_products_whose_sums_are_put_aside(plans, ta, tb):
    """In tiles of 64 with fewer ranges of k than they could have, and in place of eight ranges of tiles of 128; not where the ranges are as many as
    they can be, nor beside the kernel with one chain over all of k."""
    from test_tiles_and_scans import FOLD_KS
    # (NT: aligned where k is a multiple of 64, which the other kernel may be asked about)
    for n, k, m, folds in [(449, k, 450, True) for k in FOLD_KS if k % 64 > 0 or ta or not tb] + [(700, 700, 700, True), (3329, 4543, 190, True), (1500, 1000, 1100, False),
                                                                   (128, 896, 640, False), (211, 447, 232, False), (1024, 512, 768, False)]:
        for entry in ("plain", "multiply"):
            (_, names), = routes(plans, [(entry, n, k, m, 1, 1, ta, tb)])
            assert bool(_has(names, "gemm_tileILi3E")) == folds, (n, k, m, names)


def test_bf16_products_whose_sums_are_put_aside_for_the_ranges_that_tiles_of_128_would_have(plans):
    """Four or five against one or two of tiles of 64, which have two chains over each."""
    for n, k, m, ta, tb, folds in ((1258, 2122, 1110, 1, 0, True), (768, 2816, 1408, 0, 1, True), (256, 2688, 4480, 0, 1, True), (2128, 840, 1544, 0, 0, False)):
        (_, names), = routes(plans, [("plain", n, k, m, 1, 1, ta, tb)])
        assert bool(_has(names, "gemm_tileILi3E")) == folds, (n, k, m, names)


@pytest.mark.parametrize("ta,tb", [(0, 0), (0, 1), (1, 0), (1, 1)])
def test_bf16_products_in_two_ranges_of_tiles_of_128(plans, ta, tb):
    """... where more than 512 tiles of 64 could not be split; 512 of them and batches stay with those."""
    for n, k, m, batch, tile, ranges in ((1504, 3076, 1797, 1, 128, 2), (395, 6072, 5383, 1, 128, 2), (2047, 2500, 1023, 1, 64, 1), (232, 5030, 104, 91, 64, 1)):
        (_, names), = routes(plans, [("plain", n, k, m, batch, 1, ta, tb)], "grids")
        name, grid = names[-1].split(":")
        assert "ELi%dEEEv" % tile in name and int(grid) == -(-n // tile) * -(-m // tile) * batch * ranges, names


@pytest.mark.parametrize("n,k,m", [(5056, 64, 2176), (4288, 64, 2112)])
def test_single_products_of_short_k_whose_scans_do_not_ride(plans, n, k, m):
    """NT and TN, where one launch at most is at stake (TN 32.6 us in tiles of 256 x 256, 36.1 in tiles of 64)."""
    for ta, tb in ((0, 1), (1, 0)):
        (_, names), = routes(plans, [("protected", n, k, m, 1, 1, ta, tb)])
        assert _has(names, "gemm_bf16_256"), names
