"""k_unpack8 (layers with 8-bit words, a wave per chunk of 64 bins) at the edges of its rule: one or two
packets on tables of any size; up to 4 packets from 5120 chunks on; up to 8 from 4096 on where all such bins have
at most 40 elements, from 6144 on where they have at most 53; any number where they have at most 32, from 3072
chunks on; with the optimizer where they have at most 16.
Against the CPU oracle, bit for bit.  Needs an MI355X."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

import adacomp_workloads as W  # noqa: E402

f32 = np.float32

# bins of 1 to 64 elements, chunks that end in a short bin and in a 16-byte slot that is not full, layers of
# one to five elements, 16-bit layers among them, one of them with bins longer than an unpack tile
LAYERS = [("a", 64 * 700 + 13, 1), ("b", 1, 64), ("c", 3 * 64 * 300 + 5, 3), ("d", 500 * 70 + 3, 500), ("e", 7 * 64 * 400 + 2, 7),
          ("f", 5, 50), ("g", 50 * 64 * 90 + 49, 50), ("h", 64 * 64 * 40 + 63, 64), ("i", 5000 * 3 + 1, 5000), ("j", 2, 9)]
TABLES = {
    "small": LAYERS[1:6] + LAYERS[8:],                           # below every threshold: one or two packets only
    "5200_chunks": LAYERS + [("k", 2 * 64 * 3670 + 1, 2)],       # up to 4 packets
    # 16-bit groups that outnumber the chunks: two chunks to a workgroup (beyond L_T 26), one (beyond 53); an odd
    # number of chunks, so that the last workgroup is not full
    "few_chunks_up_to_27": [("a", 27 * 64 * 2 + 5, 27), ("b", 500 * 120 + 3, 500)],
    "few_chunks_up_to_53": [("a", 53 * 64 * 4 + 30, 53), ("b", 500 * 60 + 3, 500)],
    "few_chunks_up_to_64": [("a", 64 * 64 * 4 + 63, 64), ("b", 500 * 60 + 3, 500), ("c", 50, 50)],
    # up to 8 packets, on both sides of the two lines
    "4090_chunks_up_to_40": [("a", 2 * 64 * 4050 + 1, 2), ("b", 40 * 64 * 38 + 7, 40), ("c", 500 * 70 + 3, 500)],
    "4100_chunks_up_to_40": [("a", 2 * 64 * 4060 + 1, 2), ("b", 40 * 64 * 38 + 7, 40), ("c", 500 * 70 + 3, 500)],
    "6140_chunks_up_to_53": [("a", 2 * 64 * 6100 + 1, 2), ("b", 53 * 64 * 38 + 7, 53), ("c", 500 * 70 + 3, 500)],
    "6150_chunks_up_to_53": [("a", 2 * 64 * 6110 + 1, 2), ("b", 53 * 64 * 38 + 7, 53), ("c", 500 * 70 + 3, 500)],
    "3100_chunks_up_to_32": [l for l in LAYERS if l[2] <= 32 or l[2] > 64] + [("k", 2 * 64 * 1670 + 1, 2), ("l", 32 * 64 * 40 + 3, 32)],   # any number
    "3100_chunks_up_to_16": [l for l in LAYERS if l[2] <= 16 or l[2] > 64] + [("k", 2 * 64 * 1670 + 1, 2), ("l", 16 * 64 * 40 + 3, 16)],   # the optimizer too
}


@pytest.fixture(scope="module")
def H():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import gpu_harness
    return gpu_harness


@pytest.mark.parametrize("dense", [False, True])
@pytest.mark.parametrize("name", sorted(TABLES))
def test_sums(H, oracle_lib, name, dense):
    """1, 2, 4, 5, 8, 9, 17 and 70 packets (batches of 8 in flight, sums carried over launches of 64); dense: every
    element sent, so that bins send up to 64 words."""
    wl = W.custom(name, TABLES[name], dist="normal")
    table, n = wl.table(), wl.n_total
    chunks = sum(-(-(-(-m // lt)) // 64) for _, m, lt in table if lt <= 64)
    assert chunks < 3072 if name == "small" or name.startswith("few") else chunks >= (5120 if name == "5200_chunks" else 3072)
    mask = H.layer_mask(table, n)
    counts = (1, 2, 4, 8) if dense else (0, 1, 2, 4, 5, 8, 9, 17, 70)
    gpu = H.GpuSide(table, n, max(counts))
    try:
        cpu = []
        for k in range(max(counts)):
            g = np.random.default_rng(k).standard_normal(n).astype(f32) * f32(10.0 ** ((k % 7) - 3))
            if dense:
                g = np.where((np.arange(n) + k) % 3 == 0, -0.5, 0.5).astype(f32) * f32(k + 1)
            cpu.append(oracle_lib.compress(table, g, np.zeros(n, f32)))
            gpu.packets[k][:cpu[k].size].copy_(torch.from_numpy(cpu[k]))
        for c in counts:
            H.say(f"k_unpack8: {name}, {c} packets, dense {dense}")
            got = gpu.unpack(list(range(c)))
            want = oracle_lib.unpack_accumulate(table, cpu[:c], n)
            assert np.array_equal(got[mask].view(np.uint32), want[mask].view(np.uint32)), c
            assert np.isnan(got[~mask]).all()
    finally:
        gpu.close()


@pytest.mark.parametrize("kind,with_dense", [(1, False), (2, True)])
def test_updates(H, oracle_lib, kind, with_dense):
    import test_gpu_parity
    test_gpu_parity._update_case(oracle_lib, W.custom("unpack8_update", TABLES["3100_chunks_up_to_16"], dist="normal_outliers"), 3, 2, kind, with_dense, seed=6)


def test_packets_that_do_not_belong(H, oracle_lib):
    """A packet with a broken header, or whose words would lie past its end, contributes nothing; the others do."""
    import packet_format as pf
    wl = W.custom("broken", TABLES["5200_chunks"], dist="normal")
    table, n = wl.table(), wl.n_total
    mask = H.layer_mask(table, n)
    cpu = [oracle_lib.compress(table, W.gradient(wl, k, 0, seed=2), np.zeros(n, f32)) for k in range(3)]
    gpu = H.GpuSide(table, n, 3)
    try:
        for k in range(3):
            gpu.packets[k][:cpu[k].size].copy_(torch.from_numpy(cpu[k]))
        gpu.packets[0][0] = 0                                    # magic
        short = min(int(l["rec"]["words_offset"]) for l in pf.parse(cpu[1])[1])   # an end before the first word
        gpu.packets[1][16:24].copy_(torch.from_numpy(np.array([short], np.uint64).view(np.uint8)))
        got = gpu.unpack([0, 1, 2])
        want = oracle_lib.unpack_accumulate(table, cpu[2:], n)
        w8 = np.zeros(n, bool)
        for off, m, lt in table:
            w8[off:off + m] = lt <= 64
        assert np.array_equal(got[w8].view(np.uint32), want[w8].view(np.uint32))
        assert np.isnan(got[~mask]).all()
    finally:
        gpu.close()
