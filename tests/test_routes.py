"""Which kernels a call launches and over which grids, as the comments beside the dispatch state it; no GPU is needed."""
import pytest

from route_util import BF16, LOGIT, PROB, build_driver, routes

DENSE_F32, DENSE_BF16, SPARSE, IDENTITY = range(4)
UNITS = 256   # compute units


@pytest.fixture(scope="module")
def ask(tmp_path_factory):
    exe = build_driver(tmp_path_factory.mktemp("routes"))

    def answer(lines):
        out = routes(exe, lines)
        assert all(r.status == 0 for r in out)
        return out
    return answer


def test_splits_of_the_fp32_product_run_side_by_side(ask):
    """A product whose slots are split has no more workgroups than the chip has compute units: it would take a second round."""
    sizes = sorted({int(1000 * 64 ** (i / 80)) for i in range(81)} | {5200, 13000, 18600})
    lines, shapes = [], []
    for N in sizes:
        lines.append("kernel %d %d %d 0" % (DENSE_F32, N, min(16000, N // 3)))
        shapes.append(None)
        for B in (1, 8, 64, 65, 100, 128, 129, 192, 256):
            lines.append("exact %d %d" % (PROB, B))
            shapes.append((N, B))
    split = 0
    for shape, r in zip(shapes, ask(lines)):
        if shape is None or not any(x.kernel == "exact_reduce_kernel" for x in r.launches):
            continue
        grid = [x.grid for x in r.launches if x.kernel.startswith("exact_f32_split_kernel")]
        assert len(grid) == 1 and grid[0][0] <= UNITS, shape
        split += 1
    assert split > 300


# Column groups (128 ids) of the 16-bit product that are left after whole rounds of the chip, which holds three workgroups of two
# wavefronts on a compute unit (up to 64 positions), two of four (up to 128) and one of the larger ones: a launch of its own, its
# slots split over the chip.
@pytest.mark.parametrize("B,resident", [(64, 3), (65, 2), (128, 2), (129, 1), (256, 1), (257, 1)])
def test_last_round_of_the_16_bit_product(ask, B, resident):
    full = resident * UNITS
    for rounds in (1, 2):
        for tail in (1, 8, 92, UNITS // 2, UNITS // 2 + 1, full - 1):
            assert_cut(ask, B, rounds * full + tail, 2000, tail if tail <= UNITS // 2 else 0, full)


# Two on a unit, and half a round and some groups left: the ones after the half round, where they are few or the rows long.
@pytest.mark.parametrize("n,tail,cut", [(2000, 32, True), (7000, 32, True), (7001, 32, False), (2000, 33, False), (8999, 1, False),
                                        (9000, 1, True), (9000, 128, True), (9000, 129, False)])
def test_last_half_round_of_the_16_bit_product(ask, n, tail, cut):
    for rounds in (1, 2):
        assert_cut(ask, 100, rounds * 2 * UNITS + UNITS + tail, n, tail if cut else 0, 2 * UNITS)
    assert_cut(ask, 100, UNITS + tail, n, 0, 2 * UNITS)       # all of them run side by side


def assert_cut(ask, B, groups, n, tail, full):
    lines = ["kernel %d %d %d 0" % (DENSE_BF16, groups * 128, n)]
    lines.append("exact %d %d" % (PROB, B))
    grids = [x.grid for x in ask(lines)[1].launches if x.kernel.startswith("exact_bf16_kernel")]
    if tail:
        assert grids[0] == (groups - tail, 1, 1) and grids[1][:2] == (tail, 1) and 2 <= grids[1][2] <= full // tail, grids
    else:
        assert grids == [(groups, 1, 1)], grids


# Eq. 3 with q' written (alone and fused) and without: rows of one workgroup in one launch, and what takes the others.
WRITTEN = [(24576, 63, 3), (24577, 63, 0), (24577, 64, 3), (32768, 1024, 3), (32769, 64, 0), (32768, 1025, 1), (8192, 1025, 3),
           (8193, 1025, 1), (8192, 20000, 3), (200, 2048, 3), (2047, 2049, 0), (2048, 2049, 3), (32768, 5000, 1)]
FINISHED = [(4096, 1025, 3), (4096, 20000, 3), (5, 20000, 3), (4097, 513, 1), (4097, 1025, 1), (8192, 512, 3), (8192, 3000, 1), (8193, 257, 0),
            (12288, 256, 3), (12289, 256, 1), (32768, 256, 1), (32769, 256, 0), (32768, 1, 1)]


@pytest.mark.parametrize("N,B,kinds", WRITTEN)
def test_rows_of_eq3_written_in_one_launch(ask, N, B, kinds):
    """kinds: bit 0 = probabilities, bit 1 = logits take one launch."""
    lines = ["kernel %d %d %d 0" % (IDENTITY, N, max(4, N // 4))]
    for kind in (PROB, LOGIT, BF16):
        lines += ["linear 0 %d %d %d" % (kind, kind, B), "fused 0 %d %d %d 1" % (kind, kind, B)]
    for i, r in enumerate(ask(lines)[1:]):
        one = kinds & (1 if i < 2 else 2)
        names = [x.kernel.split("<")[0] for x in r.launches]
        assert names == ["taylor_whole_kernel"] if one else "taylor_write_kernel" in names, (i, names)


@pytest.mark.parametrize("N,B,kinds", FINISHED)
def test_rows_of_eq3_finished_in_one_launch(ask, N, B, kinds):
    lines = ["kernel %d %d %d 0" % (IDENTITY, N, max(4, N // 4))]
    lines += ["fused 0 %d %d %d 0" % (kind, kind, B) for kind in (PROB, LOGIT, BF16)]
    for i, r in enumerate(ask(lines)[1:]):
        one = kinds & (1 if i < 1 else 2)
        names = [x.kernel.split("<")[0] for x in r.launches]
        assert names == ["taylor_whole_kernel" if one else "taylor_row_kernel"], (i, names)


def test_workspace_of_rounds(ask, tmp_path):
    """Token trees of long rows: a launch a round with the workspace that the library asks for, one workgroup a position with less, and
    nothing with less than the partial statistics of the target rows take."""
    for kind in (PROB, LOGIT, BF16):
        for N, C, B, rounds in ((40000, 1, 128, 1), (39999, 1, 128, 0), (50000, 1, 129, 1), (49999, 1, 129, 0), (100000, 4, 32, 1), (200000, 1, 256, 1), (200000, 1, 257, 0)):
            r = ask(["multi %d %d %d %d -1" % (kind, B, N, C)])[0]
            names = [x.kernel.split("<")[0] for x in r.launches if x.kernel.startswith("verify")]
            assert names == ["verify_multi_round_kernel"] * (C + 1) if rounds else names == ["verify_multi_kernel"], (N, C, B, names)
            if rounds:
                less = ask(["multi %d %d %d %d %d" % (kind, B, N, C, r.workspace - 257)])[0]   # 256 of them are slack
                assert [x.kernel.split("<")[0] for x in less.launches if x.kernel.startswith("verify")] == ["verify_multi_kernel"]
    exe = build_driver(tmp_path)
    assert [r.status for r in routes(exe, ["multi %d 4 100000 1 256" % PROB, "multi %d 4 100000 1 255" % PROB])] == [0, 6]
