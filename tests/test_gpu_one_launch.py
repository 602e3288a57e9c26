"""The one-launch compress (k_pack) on tables that reach both of its forms, with and without the wait for
other workgroups succeeding, against the CPU oracle bit for bit.  Needs an MI355X."""
import contextlib

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

import adacomp_workloads as W  # noqa: E402

f32 = np.float32

# up to 16 layers and 512 tiles: every workgroup reads all records; beyond: a workgroup per layer does.
# Bin lengths from the shortest the kernel takes (4) to the longest of its tile class, slots that straddle
# bins (lengths that are no multiple of 4), both word widths, layers that end inside a 16-byte slot
FEW_LAYERS = [("a", 4 * 1025 + 3, 4), ("b", 5 * 2111 + 1, 5), ("c", 50 * 203 + 2, 50), ("d", 64 * 130 + 5, 64), ("e", 65 * 130 + 7, 65),
              ("f", 500 * 61 + 216, 500), ("g", 1023 * 9 + 1, 1023), ("h", 4096 * 3 + 9, 4096), ("i", 1, 500), ("j", 6, 7)]
TABLES = {
    "one_tile": [("a", 777, 50)],
    "few_layers": FEW_LAYERS,
    "many_layers": FEW_LAYERS + [(f"m{i}", 1 + (i * 613) % 9001, (4, 7, 50, 63, 500, 1001)[i % 6]) for i in range(60)],
    "one_long_layer": [("a", 4000 * 520 + 37, 500)],        # 521 tiles: beyond the 512 of the first form
    "two_long_layers_short_bins": [("a", 4000 * 700 + 11, 50), ("b", 4032 * 300 + 5, 64)],
}
# the longest layer that goes in one launch (four records to a thread of the workgroup that adds them up), and one
# tile more; the most layers, and one more
EDGES = {
    "512_tiles_16_layers": [(f"l{i}", 4000 * 32 - 3 * i, 500) for i in range(16)],   # the most that every workgroup reads, and half as many
    "256_tiles_16_layers": [(f"l{i}", 4000 * 16, 500 if i % 2 else 50) for i in range(16)],
    "1024_tiles": [("a", 4000 * 1023 + 5, 50)],
    "1025_tiles": [("a", 4000 * 1024 + 5, 50)],
    "1024_tiles_long_bins": [("a", 4000 * 1024 - 500, 500)],
    "512_layers": [(f"l{i}", 1 + (i * 389) % 2500, (50, 500, 9, 64)[i % 4]) for i in range(512)],
    "513_layers": [(f"l{i}", 1 + (i * 389) % 2500, (50, 500, 9, 64)[i % 4]) for i in range(513)],
}


@pytest.fixture(scope="module")
def H():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import gpu_harness
    return gpu_harness


class _Impatient:
    """Every GpuSide made inside polls once and then works out what is missing itself."""

    def __init__(self, H):
        self.H = H

    def __enter__(self):
        import paper_1712_02679_amd as A
        self.real = self.H.GpuSide

        class Side(self.real):
            def __init__(side, *args, **kw):
                super().__init__(*args, **kw)
                A.adacomp_debug_wait_polls(side.ws, 0)
        self.H.GpuSide = Side

    def __exit__(self, *exc):
        self.H.GpuSide = self.real


def layer_tiles(ws, n_layers):
    """(first tile, number of tiles) of every layer, from the layer records of an initialised workspace."""
    records = ws[256:256 + 64 * n_layers].cpu().numpy().view(np.uint32).reshape(n_layers, 16)
    return [(int(r[10]), int(r[11])) for r in records]


def tiles_of(table):
    """Compress tiles that the library makes of a table."""
    import paper_1712_02679_amd as A
    ws = torch.zeros(A.adacomp_workspace_bytes(table), dtype=torch.uint8, device="cuda")
    A.adacomp_workspace_init(table, ws)
    torch.cuda.synchronize()
    tiles = sum(layer_tiles(ws, len(table))[-1])
    A.adacomp_workspace_release(ws)
    return tiles


@pytest.mark.parametrize("name,batch,impatient", [(n, b, False) for n in sorted(TABLES) for b in (False, True)] +
                         [(n, b, True) for n in sorted(TABLES) for b in (False, True)])
def test_one_launch_tables(H, oracle_lib, name, batch, impatient):
    wl = W.custom(name, TABLES[name], dist="normal_outliers")
    say = f"one launch: {name}, batch {batch}, impatient {impatient}"
    if impatient:
        with _Impatient(H):
            H.run_parity(oracle_lib, wl, 3, 3, seed=31, label=say, batch=batch)
    else:
        H.run_parity(oracle_lib, wl, 3, 3, seed=31, label=say, batch=batch)


@pytest.mark.parametrize("name,impatient", [(n, False) for n in sorted(EDGES)] + [("1024_tiles", True), ("512_layers", True), ("512_tiles_16_layers", True)])
def test_one_launch_edges(H, oracle_lib, name, impatient):
    table = W.custom(name, EDGES[name], dist="normal_outliers").table()
    if "_tiles" in name:
        assert tiles_of(table) == int(name.split("_")[0])
    with _Impatient(H) if impatient else contextlib.nullcontext():
        H.run_parity(oracle_lib, W.custom(name, EDGES[name], dist="normal_outliers"), 2, 2, seed=32, label=f"one launch: {name}, impatient {impatient}")


@pytest.mark.parametrize("name", ["few_layers", "many_layers"])
def test_one_launch_non_finite(H, name):
    """NaN and infinite gradients in both forms: the packet keeps its structure and its length, nothing is written
    behind it or outside the layers, and what has no such gradient in its layer is what it was."""
    import packet_format as pf
    wl = W.custom(name, TABLES[name], dist="normal_outliers")
    table, n = wl.table(), wl.n_total
    mask = H.layer_mask(table, n)
    gpu, clean = H.GpuSide(table, n, 1), H.GpuSide(table, n, 1)
    try:
        rng = np.random.default_rng(405)
        off, m, _ = table[2]                       # a layer that stays finite
        for t in range(3):
            H.say(f"one launch: {name}, not finite, step {t}")
            g = W.gradient(wl, 0, t, seed=405)
            want = pf.parse(clean.compress(0, g)[:int(pf.header(clean.packets[0].cpu().numpy())["total_bytes"])], check=False)[1][2]
            bad = rng.choice(n, 400, replace=False)
            bad = bad[(bad < off) | (bad >= off + m)]
            g[bad[0::3]], g[bad[1::3]], g[bad[2::3]] = np.nan, np.inf, -np.inf
            buf = gpu.compress(0, g)
            h = pf.header(buf)
            total = int(h["total_bytes"])
            assert int(h["status"]) == 0 and total <= gpu.bound and np.all(buf[total:] == H.POISON)
            got = pf.parse(buf[:total])[1][2]
            assert got["rec"]["scale"] == want["rec"]["scale"] and got["rec"]["n_selected"] == want["rec"]["n_selected"]
            r, r_clean = gpu.residue[0].cpu().numpy(), clean.residue[0].cpu().numpy()
            assert np.all(r[~mask] == 0) and np.array_equal(r[off:off + m], r_clean[off:off + m])
    finally:
        clean.close()
        gpu.close()


@pytest.mark.parametrize("name", ["few_layers", "many_layers"])
def test_one_launch_truncated(H, oracle_lib, name):
    """A capacity in the middle of the words, in both forms: the oracle's bytes up to there, nothing past it."""
    import packet_format as pf
    import paper_1712_02679_amd as A
    wl = W.custom(name, TABLES[name], dist="normal")
    table, n = wl.table(), wl.n_total
    g, R = W.gradient(wl, 0, 0, seed=33), np.zeros(n, f32)
    want = oracle_lib.compress(table, g, R)
    fixed = A.adacomp_packet_fixed_bytes(table)
    for cap in (fixed, fixed + (want.size - fixed) // 2 // 16 * 16 + 7, want.size - 1):
        gpu = H.GpuSide(table, n, 1, capacity=cap)
        try:
            H.say(f"one launch: {name}, truncated at {cap}")
            buf = gpu.compress(0, g)
            h = pf.header(buf)
            assert h["status"] == 1 and h["total_bytes"] == want.size and np.all(buf[cap:] == H.POISON)
            same = buf[:cap] == want[:cap]
            same[8:12] = True                      # the status word itself
            if cap % 2:
                same[cap - 1] = True               # half of a 16-bit word is not written
            assert np.all(same)
            assert np.array_equal(gpu.residue[0].cpu().numpy(), R)
        finally:
            gpu.close()


@pytest.mark.parametrize("rule,factor", [(1, 2.0), (2, 2.0), (0, 1.5)])
@pytest.mark.parametrize("name,impatient", [("few_layers", False), ("many_layers", False), ("few_layers", True), ("many_layers", True)])
def test_one_launch_variants(H, oracle_lib, name, impatient, rule, factor):
    """The other rules, with gradients that hold zeros and all-zero bins (the printed compare sends those, but
    nothing that lies past a tile)."""
    wl = W.custom(name, TABLES[name], dist="normal")
    zeros = lambda k, t: (W.gradient(wl, k, t, seed=5) * ((np.arange(wl.n_total) // 97 + k) % 3 != 0)).astype(f32)
    with _Impatient(H) if impatient else contextlib.nullcontext():
        H.run_parity(oracle_lib, wl, 2, 3, grads=zeros, rule=rule, soft_factor=factor, label=f"one launch: {name} rule {rule}, impatient {impatient}",
                     batch=True)


@pytest.mark.parametrize("rule,factor", [(0, 2.0), (1, 2.0), (2, 2.0), (0, 1.5)])
@pytest.mark.parametrize("n,tiles,per", [(1, 511, 4000), (1, 512, 4000), (1, 511, 2052), (2, 255, 2048), (2, 255, 2052), (2, 256, 2052), (3, 169, 2048), (3, 170, 4000)])
def test_threads_per_tile(H, oracle_lib, n, tiles, per, rule, factor):
    """256 or 512 threads to a tile, at the line between them (512 workgroups, one per learner for the header), with
    tiles that leave the second row of slots empty (2048 elements), by one slot (2052) or not at all."""
    wl = W.custom("line", [("x", per * (tiles - 9) - 5, per), ("y", per * 9 - 1, per)], dist="normal")   # a bin to a tile
    assert tiles_of(wl.table()) == tiles
    H.run_parity(oracle_lib, wl, n, 2, rule=rule, soft_factor=factor, seed=6, label=f"one launch: {tiles} tiles of {per}, {n} learners", batch=True)


# bins of the larger tile class, of which one layer is enough for all to have such tiles: starts at every place of a
# 16-byte slot, bins that fill a tile, one element more than the class takes with its misalignment, bins of four
LARGE = [("a", 8000 * 5 + 3, 8000), ("b", 5001 * 7 + 1, 5001), ("c", 16384 * 2, 16384), ("d", 1027 * 9 + 5, 1027), ("e", 50 * 1700 + 7, 50),
         ("f", 16383 * 3 + 5, 16383), ("g", 1, 9000), ("h", 4 * 3000 + 1, 4), ("i", 4099 * 4 + 2, 4099), ("j", 65 * 300 + 3, 65)]
# tiles of 1024 bins that end inside a row of the threads' slots (of 4096 elements), and such that fill it
THOUSAND_BINS = [("a", 9000 * 3 + 1, 9000)] + [(f"t{t}", 1024 * t * (16 if t < 9 else 9) + 3 * t + 2, t) for t in (5, 6, 7, 8, 9, 10, 11, 13, 14, 15, 16)]
LARGE_TABLES = {
    "large_few_layers": LARGE,
    "large_many_layers": LARGE + [(f"m{i}", 1 + (i * 613) % 30001, (4, 7, 50, 9001, 500, 16381)[i % 6]) for i in range(40)],
    "thousand_bins_few_layers": THOUSAND_BINS,
    "thousand_bins_many_layers": THOUSAND_BINS + [(f"m{i}", 50 * i + 1, 50) for i in range(6)],
    "256_large_tiles": [("a", 16384 * 255 + 9, 16384), ("b", 50 * 900, 50)],
    "257_large_tiles": [("a", 16384 * 256 + 9, 16384), ("b", 50 * 900, 50)],
}


@pytest.mark.parametrize("n,rule,factor", [(1, 0, 2.0), (3, 0, 2.0), (2, 1, 2.0), (2, 2, 2.0), (1, 0, 1.5)])
@pytest.mark.parametrize("name,impatient", [(n, False) for n in sorted(LARGE_TABLES)] + [("large_few_layers", True), ("large_many_layers", True), ("thousand_bins_few_layers", True)])
def test_large_tiles(H, oracle_lib, name, impatient, n, rule, factor):
    wl = W.custom(name, LARGE_TABLES[name], dist="normal_outliers")
    with _Impatient(H) if impatient else contextlib.nullcontext():
        H.run_parity(oracle_lib, wl, n, 2, rule=rule, soft_factor=factor, seed=17, label=f"one launch: {name}, {n} learners, rule {rule}, impatient {impatient}",
                     batch=True)


def test_large_tiles_lazy_and_staged(H, oracle_lib, monkeypatch):
    """The staged and the lazy calls over the same tiles, in turn with one-launch ones."""
    monkeypatch.setitem(TABLES, "many_layers", LARGE_TABLES["large_many_layers"])
    test_one_launch_beside_staged_calls(H, oracle_lib)


def test_many_large_tiles_staged(H, oracle_lib):
    """More than 2048 tiles of the larger class in layers that are too long for one launch: eager and lazy."""
    wl = W.custom("long", [("a", 15000 * 1100 + 7, 5000), ("b", 16382 * 1000 - 5, 16382)], dist="normal_spikes")
    H.run_parity(oracle_lib, wl, 1, 2, seed=14, label="staged: 2100 large tiles")
    H.run_lazy_parity(oracle_lib, wl, 1, 3, 2, seed=14, label="staged, lazy: 2100 large tiles")


LAZY_TABLES = {**{n: TABLES[n] for n in ("one_tile", "few_layers", "many_layers", "two_long_layers_short_bins")},
               **{n: LARGE_TABLES[n] for n in ("large_few_layers", "large_many_layers", "thousand_bins_few_layers", "thousand_bins_many_layers")}, "512_tiles_16_layers": EDGES["512_tiles_16_layers"]}


@pytest.mark.parametrize("dense", [False, True])
@pytest.mark.parametrize("name,n,impatient", [(n, k, False) for n in sorted(LAZY_TABLES) for k in (1, 3)] +
                         [(n, 2, True) for n in ("few_layers", "many_layers", "large_few_layers", "large_many_layers")])
def test_lazy_in_one_launch(H, oracle_lib, name, n, impatient, dense):
    """Lazy calls in one launch and staged ones in turn, the corrections that one leaves applied by the other; the
    residue as the calls leave it (G everywhere) and after a sync, eager calls behind that."""
    import paper_1712_02679_amd as A
    wl = W.custom(name, LAZY_TABLES[name], dist="normal_outliers")
    table, m = wl.table(), wl.n_total
    ws = torch.zeros(A.adacomp_workspace_bytes_batch(table, n), dtype=torch.uint8, device="cuda:0")
    A.adacomp_workspace_init(table, ws)
    if impatient:
        A.adacomp_debug_wait_polls(ws, 0)
    bound = A.adacomp_packet_bound(table)
    R = [np.zeros(m, f32) for _ in range(n)]
    res = [torch.zeros(m, device="cuda:0") for _ in range(n)]
    pk = [torch.zeros(bound, dtype=torch.uint8, device="cuda:0") for _ in range(n)]
    try:
        for t in range(9):
            H.say(f"lazy in one launch: {name}, {n} learners, impatient {impatient}, dense {dense}, step {t}")
            g = [W.gradient(wl, k, t, seed=3) for k in range(n)]
            if dense:   # every element of a bin is its maximum
                g = [(np.where((np.arange(m) + k) % 3 == 0, -0.5, 0.5) * (k + 1)).astype(f32) - R[k] for k in range(n)]
            gd = [torch.from_numpy(x).cuda() for x in g]
            A.adacomp_tuning_fold_scan(t not in (2, 4, 5))   # t 2, 4, 5: staged
            before = [x.copy() for x in R]
            (A.adacomp_compress_batch if t == 7 else A.adacomp_compress_batch_lazy)(table, gd, res, pk, ws)
            torch.cuda.synchronize()
            for k in range(n):
                want = oracle_lib.compress(table, g[k], R[k])
                assert np.array_equal(pk[k][:want.size].cpu().numpy(), want), (t, k)
                left = R[k] if t == 7 else before[k] + g[k]
                mask = H.layer_mask(table, m)
                assert np.array_equal(res[k].cpu().numpy()[mask].view(np.uint32), left[mask].view(np.uint32)), (t, k)
            if t in (6, 8):
                A.adacomp_residue_sync(ws)
                torch.cuda.synchronize()
                for k in range(n):
                    assert np.array_equal(res[k].cpu().numpy(), R[k]), (t, k)
    finally:
        A.adacomp_tuning_fold_scan(True)
        A.adacomp_workspace_release(ws)


def test_one_launch_beside_staged_calls(H, oracle_lib):
    """One workspace: one-launch calls, three-launch calls (the tuning knob) and lazy calls in turn: the residues go
    on as if nothing had changed."""
    import paper_1712_02679_amd as A
    wl = W.custom("turns", TABLES["many_layers"], dist="normal")
    table, n = wl.table(), wl.n_total
    ws1 = torch.zeros(A.adacomp_workspace_bytes_batch(table, 2), dtype=torch.uint8, device="cuda:0")
    A.adacomp_workspace_init(table, ws1)
    bound = A.adacomp_packet_bound(table)
    R = [np.zeros(n, f32) for _ in range(2)]
    res = [torch.zeros(n, device="cuda:0") for _ in range(2)]
    pk = [torch.zeros(bound, dtype=torch.uint8, device="cuda:0") for _ in range(2)]
    try:
        for t in range(8):
            g = [W.gradient(wl, k, t, seed=3) for k in range(2)]
            gd = [torch.from_numpy(x).cuda() for x in g]
            kind = t % 4
            A.adacomp_tuning_fold_scan(kind != 1)
            if kind == 2:
                A.adacomp_compress_batch_lazy(table, gd, res, pk, ws1)
                A.adacomp_residue_sync(ws1)
            elif kind == 3:
                for k in range(2):
                    A.adacomp_compress(table, gd[k], res[k], pk[k], ws1)
                    torch.cuda.synchronize()
            else:
                A.adacomp_compress_batch(table, gd, res, pk, ws1)
            torch.cuda.synchronize()
            for k in range(2):
                want = oracle_lib.compress(table, g[k], R[k])
                assert np.array_equal(pk[k][:want.size].cpu().numpy(), want), (t, k)
                assert np.array_equal(res[k].cpu().numpy(), R[k]), (t, k)
    finally:
        A.adacomp_tuning_fold_scan(True)
        A.adacomp_workspace_release(ws1)


def test_workspace_without_room_for_exchange_areas(H, oracle_lib):
    """The least a call needs is what it was before there were exchange areas: such a workspace is accepted and
    takes the staged launches, with the same results."""
    import paper_1712_02679_amd as A
    wl = W.custom("least", TABLES["few_layers"], dist="normal")
    table, n = wl.table(), wl.n_total
    areas = A.adacomp_workspace_bytes_batch(table, 2) - A.adacomp_workspace_bytes(table) - A.adacomp_workspace_gmax(table)[2]
    assert areas > 0
    ws = torch.zeros(A.adacomp_workspace_bytes(table) - areas, dtype=torch.uint8, device="cuda:0")
    A.adacomp_workspace_init(table, ws)
    g = W.gradient(wl, 0, 0, seed=9)
    R, res = np.zeros(n, f32), torch.zeros(n, device="cuda:0")
    pk = torch.zeros(A.adacomp_packet_bound(table), dtype=torch.uint8, device="cuda:0")
    A.adacomp_compress(table, torch.from_numpy(g).cuda(), res, pk, ws)
    torch.cuda.synchronize()
    want = oracle_lib.compress(table, g, R)
    assert np.array_equal(pk[:want.size].cpu().numpy(), want) and np.array_equal(res.cpu().numpy(), R)
    A.adacomp_workspace_release(ws)


@pytest.mark.parametrize("name", ["few_layers", "many_layers"])
@pytest.mark.parametrize("areas", [0, 1, 2])
def test_more_learners_than_exchange_areas(H, oracle_lib, name, areas):
    """A workspace that accepts 3 learners and has exchange areas for fewer: a captured call of one learner,
    replayed after calls of 2 and 3 learners, staged and lazy ones among them (their scratch blocks are the
    largest that the workspace takes)."""
    import paper_1712_02679_amd as A
    wl = W.custom(name, TABLES[name], dist="normal_outliers")
    table, n = wl.table(), wl.n_total
    stride = A.adacomp_workspace_gmax(table)[2]
    area = A.adacomp_workspace_bytes_batch(table, 2) - A.adacomp_workspace_bytes(table) - stride
    assert 0 < area < stride // 3
    ws = torch.zeros(A.adacomp_workspace_bytes(table) - area + 2 * stride + areas * area, dtype=torch.uint8, device="cuda:0")
    A.adacomp_workspace_init(table, ws)
    bound = A.adacomp_packet_bound(table)
    R = [np.zeros(n, f32) for _ in range(3)]
    res = [torch.zeros(n, device="cuda:0") for _ in range(3)]
    pk = [torch.zeros(bound, dtype=torch.uint8, device="cuda:0") for _ in range(3)]
    gd = [torch.zeros(n, device="cuda:0") for _ in range(3)]
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=torch.cuda.Stream()):
        A.adacomp_compress(table, gd[0], res[0], pk[0], ws)
    try:
        for t in range(8):
            g = [W.gradient(wl, k, t, seed=8) for k in range(3)]
            for k in range(3):
                gd[k].copy_(torch.from_numpy(g[k]))
            live = 1 if t % 2 == 0 else (3, 2, 3, 3)[t // 2]
            H.say(f"exchange areas {areas}, {name}, call {t} of {live}")
            if t % 2 == 0:
                torch.cuda.synchronize()
                graph.replay()
            elif t == 5:
                A.adacomp_compress_batch_lazy(table, gd, res, pk, ws)
                A.adacomp_residue_sync(ws)
            else:
                A.adacomp_compress_batch(table, gd[:live], res[:live], pk[:live], ws)
            torch.cuda.synchronize()
            for k in range(live):
                want = oracle_lib.compress(table, g[k], R[k])
                assert np.array_equal(pk[k][:want.size].cpu().numpy(), want), (t, k)
                assert np.array_equal(res[k].cpu().numpy(), R[k]), (t, k)
    finally:
        A.adacomp_workspace_release(ws)


def test_more_workgroups_than_are_resident(H, oracle_lib):
    """A table that every workgroup could read as a whole, with so many learners that a workgroup per layer does."""
    wl = W.custom("crowd", [("a", 600 * 1000 + 3, 50), ("b", 55 * 1000 + 9, 500)], dist="normal")
    H.run_parity(oracle_lib, wl, 9, 2, seed=13, label="one launch: 9 learners", batch=True)


@pytest.mark.parametrize("odd", [0, 1])
def test_both_forms_write_the_words_of_an_area(H, odd):
    """Calls of 1 and of 9 learners on one workspace take the two forms, which share what a learner's exchange area has
    for its tiles, four words each.  The second and third, where records keep 17 bits of the call's number beside a word
    count, are written in every call; the others tell calls apart by 32 bits."""
    import paper_1712_02679_amd as A
    wl = W.custom("crowd", [("a", 600 * 1000 + 2600 * odd, 50), ("b", 55 * 1000 + 9, 500)], dist="normal")
    table, n = wl.table(), wl.n_total
    gpu = H.GpuSide(table, n, 9, batch=True)
    try:
        tiles = sum(layer_tiles(gpu.ws, len(table))[-1])   # the last layer's first tile, and how many it has
        assert tiles % 2 == odd
        area = A.adacomp_workspace_bytes_batch(table, 2) - A.adacomp_workspace_bytes(table) - A.adacomp_workspace_gmax(table)[2]
        at = gpu.ws.numel() // 128 * 128 - 9 * area + -(-16 * tiles // 128) * 128
        for call, live in enumerate((9, 1, 9, 9, 1, 1, 9)):
            g = [torch.from_numpy(W.gradient(wl, k, call, seed=2)).cuda() for k in range(live)]
            A.adacomp_compress_batch(table, g, gpu.residue[:live], gpu.packets[:live], gpu.ws, packet_capacity=gpu.capacity)
            torch.cuda.synchronize()
            words = gpu.ws[at:at + 32 * tiles].cpu().numpy().view(np.uint64).reshape(tiles, 4)
            assert np.all(words[:, 1:3] & 0x1FFFF == call + 1), (call, live)
            whole = (0, 3) if live == 1 else (0, 1, 2)
            assert np.all(words[:, whole] & 0xFFFFFFFF == call + 1), (call, live)
    finally:
        gpu.close()


@pytest.mark.parametrize("n", [33, 40])
def test_more_learners_than_a_launch(H, oracle_lib, n):
    """Calls of more than 32 learners take several launches, which use the same exchange areas in turn."""
    wl = W.custom("few_layers", TABLES["few_layers"][2:6], dist="normal")
    H.run_parity(oracle_lib, wl, n, 2, seed=12, label=f"one launch: {n} learners", batch=True)


def _masked_stream(units):
    """A stream that may use the first `units` compute units only."""
    import ctypes
    hip = ctypes.CDLL("libamdhip64.so")
    words = (ctypes.c_uint32 * 8)(*[((1 << 32) - 1 if 32 * (i + 1) <= units else 0) for i in range(8)])
    stream = ctypes.c_void_p()
    rc = hip.hipExtStreamCreateWithCUMask(ctypes.byref(stream), 8, words)
    assert rc == 0, rc
    return torch.cuda.ExternalStream(stream.value)


@pytest.mark.parametrize("name", ["few_layers", "one_long_layer", "two_long_layers_short_bins"])
@pytest.mark.parametrize("units", [32, 64])
def test_captured_call_replayed_on_few_compute_units(H, oracle_lib, name, units):
    """Captured where the whole GPU was there, replayed on a stream where the tiles of a layer do not fit: the
    workgroups that run work out the records of those that cannot start."""
    import paper_1712_02679_amd as A
    wl = W.custom(name, TABLES[name], dist="normal_outliers")
    table, n = wl.table(), wl.n_total
    ws = torch.zeros(A.adacomp_workspace_bytes(table), dtype=torch.uint8, device="cuda:0")
    A.adacomp_workspace_init(table, ws)
    pk = torch.zeros(A.adacomp_packet_bound(table), dtype=torch.uint8, device="cuda:0")
    res, gd, R = torch.zeros(n, device="cuda:0"), torch.zeros(n, device="cuda:0"), np.zeros(n, f32)
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=torch.cuda.Stream()):
        A.adacomp_compress(table, gd, res, pk, ws)
    masked = _masked_stream(units)
    try:
        for t in range(4):
            H.say(f"one launch: {name} replayed on {units} compute units, step {t}")
            g = W.gradient(wl, 0, t, seed=15)
            gd.copy_(torch.from_numpy(g))
            torch.cuda.synchronize()
            with torch.cuda.stream(masked if t != 2 else torch.cuda.current_stream()):
                graph.replay()
            torch.cuda.synchronize()
            want = oracle_lib.compress(table, g, R)
            assert np.array_equal(pk[:want.size].cpu().numpy(), want), t
            assert np.array_equal(res.cpu().numpy(), R), t
    finally:
        A.adacomp_workspace_release(ws)


@pytest.mark.parametrize("name", ["many_layers", "one_long_layer"])
@pytest.mark.parametrize("units", [32, 64])
def test_stream_with_few_compute_units(H, oracle_lib, name, units):
    """A table whose tiles do not fit the compute units of the stream takes the staged launches there."""
    wl = W.custom(name, TABLES[name], dist="normal")
    with torch.cuda.stream(_masked_stream(units)):
        H.run_parity(oracle_lib, wl, 2, 2, seed=14, label=f"one launch: {name} on {units} compute units", batch=True)
        torch.cuda.synchronize()


@pytest.mark.parametrize("name", ["few_layers", "many_layers"])
def test_one_launch_in_a_graph(H, oracle_lib, name):
    """Captured and replayed five times with eager calls in between: every replay counts on."""
    import paper_1712_02679_amd as A
    wl = W.custom(name, TABLES[name], dist="normal_outliers")
    table, n = wl.table(), wl.n_total
    ws = torch.zeros(A.adacomp_workspace_bytes(table), dtype=torch.uint8, device="cuda:0")
    A.adacomp_workspace_init(table, ws)
    pk = torch.zeros(A.adacomp_packet_bound(table), dtype=torch.uint8, device="cuda:0")
    res, gd, R = torch.zeros(n, device="cuda:0"), torch.zeros(n, device="cuda:0"), np.zeros(n, f32)
    stream = torch.cuda.Stream()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=stream):
        A.adacomp_compress(table, gd, res, pk, ws)
    for t in range(10):
        g = W.gradient(wl, 0, t, seed=4)
        gd.copy_(torch.from_numpy(g))
        torch.cuda.synchronize()
        if t % 2 == 0:
            graph.replay()
        else:
            A.adacomp_compress(table, gd, res, pk, ws)
        torch.cuda.synchronize()
        want = oracle_lib.compress(table, g, R)
        assert np.array_equal(pk[:want.size].cpu().numpy(), want), t
        assert np.array_equal(res.cpu().numpy(), R), t
    A.adacomp_workspace_release(ws)
