"""The unpack kernels that apply an optimizer step, on both sides of the line from which on they fetch weights and moments
ahead of the adds: by elements, elements to a tile, packets and word widths.  Against the CPU oracle, bit for bit.  Needs an
MI355X."""
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

import adacomp_workloads as W  # noqa: E402

# full tiles and half-empty ones; tiles that start off the 16-byte grid; a last slot that is not whole, layers that are
# none; bins cut into slices
TABLES = {
    "words16": [("a", 500 * 2400 + 217, 500), ("b", 1023 * 400 + 1, 1023), ("c", 9001 * 9 + 3, 9001), ("d", 2, 500)],
    "words16_half_empty": [("a", 65 * 23100 + 7, 65), ("b", 1, 65)],
    "words8": [("a", 50 * 24000 + 17, 50), ("b", 61 * 6000 + 2, 61), ("c", 3, 64)],
    "both": [("a", 50 * 16000 + 17, 50), ("b", 257 * 3300 + 3, 257), ("c", 5003 * 9 + 1, 5003)],
    "below_the_line": [("a", 50 * 5000 + 17, 50), ("b", 257 * 900 + 3, 257), ("c", 5003 * 9 + 1, 5003)],
}


@pytest.fixture(scope="module")
def H():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import gpu_harness
    return gpu_harness


@pytest.mark.parametrize("kind,n,with_dense", [(1, 1, False), (2, 4, True), (1, 5, True), (2, 8, False), (1, 9, True), (2, 16, False), (1, 17, False)])
@pytest.mark.parametrize("name", sorted(TABLES))
def test_updates(H, oracle_lib, name, kind, n, with_dense):
    import test_gpu_parity
    H.say(f"update: {name}, kind {kind}, {n} packets")
    test_gpu_parity._update_case(oracle_lib, W.custom(name, TABLES[name], dist="normal_outliers"), n, 1, kind, with_dense, seed=21)
