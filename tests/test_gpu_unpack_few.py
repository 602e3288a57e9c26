"""The three forms of the unpack kernel by number of packets (up to 4, up to 8, more), each for 16-bit words, 8-bit
words and tables of both, at the edges of their tiles.  Against the CPU oracle, bit for bit.  Needs an MI355X."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

import adacomp_workloads as W  # noqa: E402

f32 = np.float32

TABLES = {
    # the shortest and longest bins that share a tile, one bin to a tile, bins cut into slices; ragged ends; chunks whose last
    # tile is not full; runs of tiles end at chunk borders
    "words16": [("a", 65 * 64 * 3 + 7, 65), ("b", 500 * 77 + 216, 500), ("c", 1023 * 70 + 1, 1023), ("d", 4096 * 3 + 9, 4096), ("e", 9001 * 3 + 5, 9001),
                ("f", 16384 * 2, 16384), ("g", 1, 500), ("h", 257 * 16 * 5 + 3, 257)],
    "words8": [("a", 50 * 64 * 9 + 17, 50), ("b", 64 * 64 * 3 + 63, 64), ("c", 7 * 64 * 5 + 1, 7), ("d", 3, 64), ("e", 64 * 21 + 5, 1)],
    "both": [("a", 50 * 64 * 9 + 17, 50), ("b", 500 * 77 + 216, 500), ("c", 64 * 64 * 3 + 63, 64), ("d", 5000 * 3 + 1, 5000), ("e", 3, 9)],
    "both_in_runs": [("a", 50 * 64 * 30 + 3, 50), ("b", 500 * 64 * 300 + 123, 500), ("c", 9001 * 40, 9001)],   # some tiles of a chunk to a workgroup
    "hundreds_of_chunks": [("a", 8 * 64 * 850 + 3, 8), ("b", 500 * 64 * 6 + 123, 500)],   # up to 2 packets: a wave per chunk, and 16-bit groups in its launch
}
COUNTS = (1, 2, 3, 4, 5, 8, 9, 16, 17)


@pytest.fixture(scope="module")
def H():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import gpu_harness
    return gpu_harness


@pytest.mark.parametrize("dense", [False, True])
@pytest.mark.parametrize("name", sorted(TABLES))
def test_sums(H, oracle_lib, name, dense):
    """dense: every element sent, so that bins have more words than lanes; the last packet but one is broken in
    calls of three and five."""
    wl = W.custom(name, TABLES[name], dist="normal")
    table, n = wl.table(), wl.n_total
    mask = H.layer_mask(table, n)
    gpu = H.GpuSide(table, n, max(COUNTS))
    try:
        cpu = []
        for k in range(max(COUNTS)):
            g = np.random.default_rng(k).standard_normal(n).astype(f32) * f32(10.0 ** ((k % 7) - 3))
            if dense:
                g = np.where((np.arange(n) + k) % 3 == 0, -0.5, 0.5).astype(f32) * f32(k + 1)
            cpu.append(oracle_lib.compress(table, g, np.zeros(n, f32)))
            gpu.packets[k][:cpu[k].size].copy_(torch.from_numpy(cpu[k]))
        for c in COUNTS:
            H.say(f"unpack: {name}, {c} packets, dense {dense}")
            broken = c - 2 if c in (3, 5) else -1
            if broken >= 0:
                gpu.packets[broken][0] = 0
            got = gpu.unpack(list(range(c)))
            if broken >= 0:
                gpu.packets[broken][0] = int(cpu[broken][0])
            want = oracle_lib.unpack_accumulate(table, [p for k, p in enumerate(cpu[:c]) if k != broken], n)
            assert np.array_equal(got[mask].view(np.uint32), want[mask].view(np.uint32)), c
            assert np.isnan(got[~mask]).all()
    finally:
        gpu.close()


@pytest.mark.parametrize("kind,n,with_dense", [(1, 1, False), (2, 4, True), (1, 5, True), (2, 8, False), (1, 9, False), (2, 2, False)])
@pytest.mark.parametrize("name", ["words16", "words8", "both"])
def test_updates(H, oracle_lib, name, kind, n, with_dense):
    import test_gpu_parity
    test_gpu_parity._update_case(oracle_lib, W.custom(name, TABLES[name], dist="normal_outliers"), n, 2, kind, with_dense, seed=6)
