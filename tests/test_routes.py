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
