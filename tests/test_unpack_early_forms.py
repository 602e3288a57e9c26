"""Every form of the unpack kernels that asks for weights and moments ahead of the adds: both optimizers, both word widths and both
in one launch, up to 2, 4, 8 and 16 packets; and beside them the same calls on tables whose tiles are too empty for it.  That a case
is on its side of the line is checked without a GPU, the results against the CPU oracle, bit for bit, on an MI355X."""
import ctypes

import pytest

torch = pytest.importorskip("torch")

import adacomp_workloads as W  # noqa: E402

SGD, ADAM = 1, 2
TABLES = {
    # full tiles, of which some start off the 16-byte grid; a last slot that is not whole; bins cut into slices
    "full16": [("a", 500 * 2400 + 217, 500), ("b", 1023 * 400 + 1, 1023), ("c", 9001 * 9 + 3, 9001), ("d", 2, 500)],
    "full8": [("a", 50 * 24000 + 17, 50), ("b", 61 * 6000 + 2, 61), ("c", 3, 64)],
    "full_both": [("a", 61 * 9000 + 5, 61), ("b", 500 * 1600 + 123, 500), ("c", 1023 * 300 + 1, 1023), ("d", 3, 9)],
    # a third of a tile's room, and half of it in 16-bit layers
    "small8": [("a", 18 * 90000 + 7, 18)],
    "small_both": [("a", 20 * 50000 + 3, 20), ("b", 65 * 10000 + 7, 65)],
}
ALL = [(kind, n) for kind in (SGD, ADAM) for n in (1, 2, 3, 4, 8)]
CASES = [(name, kind, n, True) for name in ("full16", "full8", "full_both") for kind, n in ALL]
CASES += [("full16", kind, n, True) for kind in (SGD, ADAM) for n in (9, 16)]
CASES += [(name, kind, n, early) for name, behind in (("small8", (1, 2, 8)), ("small_both", (2, 8))) for kind, n, early in
          [(ADAM, 3, True), (ADAM, 4, True), (SGD, 4, True)] + [(kind, n, False) for kind in (SGD, ADAM) for n in behind]]
# beyond 64 packets the last launch adds to what the first left in dense_out: 2, 4 and 8 packets in it
CASES += [("full16", SGD, 66, True), ("full_both", ADAM, 68, True), ("full8", SGD, 72, True)]


def counts(layers, of8):
    """Elements, bins and unpack tiles of the layers with 8-bit words (True), 16-bit ones (False) or all (None)."""
    elems = bins = tiles = 0
    for _, n, lt in layers:
        if of8 is not None and (lt <= 64) != of8:
            continue
        elems, bins = elems + n, bins + -(-n // lt)
        if lt <= 4096:
            per = 1
            while per < 64 and 2 * per * lt <= 4096:
                per *= 2
            tiles += -(-(-(-n // lt)) // per)
        else:
            tiles += n // lt * -(-lt // 4096) + -(-(n % lt) // 4096)
    return elems, bins, tiles


@pytest.mark.parametrize("name,kind,n,early", CASES)
def test_cases_are_on_their_side_of_the_line(name, kind, n, early):
    import paper_1712_02679_amd as A
    rule = A.binding.lib()["_ZN7adacomp16unpack_early_forEmmmbjj"]
    rule.restype = ctypes.c_bool
    layers = TABLES[name]
    elems8, (elems, bins, tiles) = counts(layers, True)[0], counts(layers, None)
    last = (n - 1) % 64 + 1
    words8 = 3 * elems8 >= elems if 0 < elems8 < elems else elems8 == elems
    u64, u32 = ctypes.c_uint64, ctypes.c_uint32
    assert rule(u64(elems), u64(bins), u64(tiles), ctypes.c_bool(words8), u32(last), u32(kind)) == early


@pytest.mark.gpu
@pytest.mark.parametrize("name,kind,n,early", CASES)
def test_updates(oracle_lib, name, kind, n, early):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import gpu_harness as H
    import test_gpu_parity
    H.say(f"update: {name}, kind {kind}, {n} packets, {'ahead of' if early else 'behind'} the adds")
    test_gpu_parity._update_case(oracle_lib, W.custom(name, TABLES[name], dist="normal_outliers"), n, 1, kind, n % 2 == 0 or n > 64, seed=23, threads=8)
