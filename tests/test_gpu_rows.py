"""The layer kernel on fp32 rows (k_layer_seg, widths up to 16384 past the LDS tiles) against the oracle: one
and two LDS segments at their edges, the split of a column's sources between the segments, shared
outputs for few rows, and the ways its rows come from and go to the tile kernels."""
from __future__ import annotations

import gc

import numpy as np
import pytest

import oracle
from tests.gpu_util import GpuNet, assert_parity, log, oracle_run

pytestmark = pytest.mark.gpu

CAP = 10112  # sources of one LDS segment


def run(n, layers, y0):
    gpu = GpuNet(n, len(layers))
    for l, (cp, ri, v, b) in enumerate(layers):
        gpu.load(l, cp, ri, v, b)
    cats = gpu.run(y0)
    o = oracle_run(y0, layers)
    assert_parity(gpu, o, cats)
    return gpu, cats


def csc(rng, n, columns, scale):
    """A layer of the given columns (each a set of sources)."""
    cp = np.zeros(n + 1, np.int64)
    cp[1:] = np.cumsum([len(c) for c in columns])
    ri = np.concatenate([np.sort(np.asarray(c, np.int32)) for c in columns] + [np.empty(0, np.int32)]).astype(np.int32)
    return cp, ri, (rng.random(ri.size) * scale).astype(np.float32)


def layer(rng, n, kind):
    if kind == "ragged":  # any number of sources, none and one among them
        deg = rng.integers(0, 49, size=n)
        deg[:3] = (0, 1, 100)
        cols = [rng.choice(n, size=d, replace=False) for d in deg]
        scale = 0.16
    elif kind == "one-sided":  # every source at one end: no cut of 16 and 16 exists
        cols = [rng.choice(min(n, 600), size=32, replace=False) + (n - min(n, 600) if j % 2 else 0) for j in range(n)]
        scale = 0.125
    else:
        cols = [rng.choice(n, size=32, replace=False) for _ in range(n)]
        scale = 0.125
    cp, ri, v = csc(rng, n, cols, scale)
    return cp, ri, v, rng.uniform(-0.45, -0.35, size=n).astype(np.float32)


@pytest.mark.parametrize("n,m,kind", [
    (4097, 261, "ragged"), (5001, 1, "ragged"), (CAP - 1, 1100, "random"), (CAP, 270, "one-sided"),
    (CAP + 1, 1030, "random"), (CAP + 1, 3, "ragged"), (12288, 1029, "ragged"), (16383, 300, "one-sided"),
    (16384, 1301, "random"), (16384, 1, "ragged"),
])
def test_rows_layers(n, m, kind):
    """Three layers from real-valued inputs: layer 0 from the caller's rows, the others from the rows before
    (or, with 256 rows and fewer and 32 sources per column, from tiles). Rows of several densities,
    so that some die at every layer and the live rows move; 4-row groups that do not divide the rows."""
    rng = np.random.default_rng(n + m)
    dens = rng.uniform(0.35, 1.0, size=(m, 1))
    y0 = ((rng.random((m, n)) < dens) * rng.random((m, n))).astype(np.float32)
    if m > 2:
        y0[m // 2] = 0.0
    log(f"rows n={n} m={m} {kind}")
    layers = [layer(rng, n, kind) for _ in range(3)]
    gpu, cats = run(n, layers, y0)
    live = gpu.net.live_counts()
    names = gpu.net.layer_kernels()
    assert names[0] == "k_layer_seg"
    few = False  # once in tiles, layers of 32 sources stay there
    for l in (1, 2):
        few = few or (kind != "ragged" and live[l] <= 256)
        assert names[l] == ("none" if live[l] == 0 else "k_layer_gfm_small" if few else "k_layer_seg")


@pytest.mark.parametrize("n,where", [(4200, "first"), (CAP, "spread"), (CAP + 1, "first"), (16384, "last"), (16384, "spread")])
def test_rows_longest_column(n, where):
    """A column of 4096 sources, the most that the interface takes, beside columns of up to 8: one segment, and two
    with all of its sources in one of them or in both."""
    rng = np.random.default_rng(n)
    deg = rng.integers(0, 9, size=n)
    cols = [rng.choice(n, size=d, replace=False) for d in deg]
    cols[n // 3] = {"first": np.arange(4096), "last": np.arange(n - 4096, n),
                    "spread": rng.choice(n, size=4096, replace=False)}[where]
    cp, ri, v = csc(rng, n, cols, 0.3)
    v[cp[n // 3]:cp[n // 3 + 1]] *= np.float32(0.002)  # its sum stays below the upper limit
    y0 = rng.random((6, n)).astype(np.float32)
    log(f"rows, longest column n={n} {where}")
    run(n, [(cp, ri, v, np.full(n, -0.2, np.float32))], y0)


@pytest.mark.parametrize("seq", [(32, 40, 32), (40, 32, 40), (40, 40, 32)])
@pytest.mark.parametrize("m", [90, 700])
def test_rows_between_tiles(seq, m):
    """Layers of 32 and of up to 40 sources in turn: few rows go from tiles (32 sources) to rows (any other
    number) and back, more rows from one-byte codes (binary inputs, 32 sources in layer 0) to rows."""
    n = 6000
    rng = np.random.default_rng(m + seq[0])
    layers = []
    for k in seq:
        cols = [rng.choice(n, size=int(rng.integers(8, k + 1)), replace=False) for _ in range(n)]
        cols[7] = rng.choice(n, size=k, replace=False)
        cp, ri, v = csc(rng, n, cols, 0.18)
        layers.append((cp, ri, v, np.full(n, -0.3, np.float32)))
    y0 = (rng.random((m, n)) < rng.uniform(0.2, 0.7, size=(m, 1))).astype(np.float32)
    log(f"rows between tiles {seq} m={m}")
    gpu, cats = run(n, layers, y0)
    assert 0 < cats.size
    live = gpu.net.live_counts()
    assert live[2] > 256 or m == 90
    few = "k_layer_gfm_small" if m == 90 else "k_layer_seg"
    expect = ["k_pack_bits+k_layer_bits" if seq[0] == 32 else "k_layer_seg"]
    assert gpu.net.layer_kernels() == expect + ["k_layer_seg" if k == 40 else few for k in seq[1:]]


def test_rows_to_codes_and_back():
    """2,500 rows whose layer outputs are many values (rows), then one value (the encoder reads them as tiles
    and the layer gathers codes), then many again: rows to tiles to codes to rows."""
    n, m = 6000, 2500
    rng = np.random.default_rng(3)
    layers = [layer(rng, n, "random") for _ in range(4)]
    layers[1] = (*layers[1][:3], np.full(n, 40.0, np.float32))  # every output 32
    cp, ri, v, b = layers[2]
    layers[2] = (cp, ri, v * np.float32(0.25), b)  # 32 inputs of 32 sum to 16 on average: not saturated
    y0 = (rng.random((m, n)) * 2).astype(np.float32)
    gpu, cats = run(n, layers, y0)
    from paper_1909_05631_amd import sdnn
    kinds = [sdnn.KERNEL_KINDS[int(k)] for k in gpu.net.layer_info()[0]]
    assert kinds == ["k_layer_gfm", "k_layer_gfm", "k_layer_gfm_u8", "k_layer_gfm"]
    assert gpu.net.layer_kernels() == ["k_layer_seg", "k_layer_seg", "k_layer_gfm_u8", "k_layer_seg"]
    assert cats.size == m


@pytest.mark.parametrize("equal", [False, True])
@pytest.mark.parametrize("n,m,nl", [(6000, 300, 2), (6000, 300, 3), (6000, 300, 6), (6000, 700, 5), (40000, 300, 5)])
def test_codes_to_few_rows(n, m, nl, equal):
    """Binary inputs whose live rows fall to at most 256 in layer 0, which wrote codes: the layer that reads the
    codes of few rows counts its live rows, and those after it go on from its outputs."""
    rng = np.random.default_rng(n + m)
    dens = np.where(rng.random((m, 1)) < 200 / m, 0.6, 0.002)
    y0 = (rng.random((m, n)) < dens).astype(np.float32)
    layers = []
    for l in range(nl):
        cp, src, v, b = offset_layer(rng, n, -0.3)
        layers.append((cp, src, np.full_like(v, 1.0 / 16.0), b))
    log(f"codes to few rows n={n} m={m} layers={nl} equal={equal}")
    gpu = GpuNet(n, nl, equal_values=equal)
    for l, layer_ in enumerate(layers):
        gpu.load(l, *layer_)
    cats = gpu.run(y0)
    o = oracle_run(y0, layers)
    assert 0 < oracle.padded_live_counts(o, nl)[1] <= 256
    kinds = gpu.net.layer_info()[0]
    assert kinds[0] in (6, 7) and kinds[1] == 3  # codes written and read
    assert_parity(gpu, o, cats)


def test_two_handles_in_turn():
    """Two networks of one width on one stream keep their own rows and maps."""
    n, m = 9000, 600
    rng = np.random.default_rng(9)
    nets = []
    for i in range(2):
        layers = [layer(rng, n, "random") for _ in range(2)]
        y0 = rng.random((m, n)).astype(np.float32)
        gpu = GpuNet(n, 2)
        for l, (cp, ri, v, b) in enumerate(layers):
            gpu.load(l, cp, ri, v, b)
        nets.append((gpu, layers, y0))
    for gpu, layers, y0 in nets + nets[::-1]:
        cats = gpu.run(y0)
        assert_parity(gpu, oracle_run(y0, layers), cats)


def offset_layer(rng, n, bias):
    """32 sources per column: distinct offsets under two permutations."""
    off = rng.choice(n, size=32, replace=False)
    p, q = rng.permutation(n), rng.permutation(n)
    src = np.sort(p[(q[:, None] + off[None, :]) % n], axis=1).astype(np.int32)
    v = rng.uniform(0.02, 0.11, size=src.size).astype(np.float32)
    return np.arange(n + 1, dtype=np.int64) * 32, src.reshape(-1), v, np.full(n, bias, np.float32)


@pytest.mark.parametrize("n,m,nl", [
    (32, 70, 3), (36, 1, 130), (100, 300, 66), (1000, 64, 65), (1024, 9000, 5), (1028, 1100, 64), (1030, 600, 4),
    (2052, 4500, 4), (4092, 2100, 4), (4096, 260, 70), (1024, 5, 13), (1024, 5, 14), (1092, 470, 20), (1092, 498, 20),
    (1096, 3, 20),
])
def test_lds_widths_lists(n, m, nl):
    """Widths staged in LDS with 32 sources per column and per-edge weights (lists loaded a round ahead): rounds
    that the width does not fill, one row and more, tiles and 4-row groups the rows do not fill,
    depths around the 64 layers after which the fused launch adds its counts, rows that die early and
    late; depths, widths and batches on both sides of the rule for workgroups that fetch lists ahead."""
    rng = np.random.default_rng(n + nl)
    dens = rng.uniform(0.2, 0.9, size=(m, 1))
    y0 = ((rng.random((m, n)) < dens) * rng.uniform(0.2, 1.0, size=(m, n))).astype(np.float32)
    if m > 2:
        y0[1] = 0.0
    layers = [offset_layer(rng, n, -0.30) for _ in range(min(nl, 8))]
    layers = [layers[l % len(layers)] for l in range(nl)]
    if nl > 60:  # every row but the strongest dies at layer 60
        layers[60] = (*layers[60][:3], np.full(n, -58.0, np.float32))
    log(f"LDS widths, lists ahead: n={n} m={m} layers={nl}")
    gpu, cats = run(n, layers, y0)
    names = gpu.net.layer_kernels()
    if m <= 1024:
        assert names == ["k_layers_lds32"] * nl
    else:
        one = "k_layer_lds32" if n % 4 == 0 and n > 448 else "k_layer_lds"
        assert names[0] == one and set(names) <= {one, "k_layers_lds32", "none"}


@pytest.mark.parametrize("n,m,ahead", [
    (128, 1100, False), (132, 8192, True), (132, 8193, False), (192, 8193, False), (196, 65537, True), (256, 65536, False),
    (256, 65537, True), (260, 16384, False), (320, 16385, True), (324, 8193, False), (448, 12288, False), (452, 8193, True),
])
def test_lds_widths_either_kernel(n, m, ahead):
    """Both sides of the rule by width and rows between the per-layer kernels with one and two workgroups per
    CU (256 CUs, 32 rows a tile)."""
    rng = np.random.default_rng(n + m)
    y0 = ((rng.random((m, n)) < rng.uniform(0.2, 0.9, size=(m, 1))) * rng.random((m, n))).astype(np.float32)
    log(f"LDS widths, either kernel: n={n} m={m}")
    gpu, cats = run(n, [offset_layer(rng, n, -0.30) for _ in range(3)], y0)
    assert gpu.net.layer_kernels()[0] == ("k_layer_lds32" if ahead else "k_layer_lds")


@pytest.mark.parametrize("n,m", [(64, 9000), (1024, 9000), (2048, 4500), (4096, 2300)])
def test_lds_widths_nonzero_inputs_of_one_wave(n, m):
    """Every row has one nonzero input, at a neuron that the first or the last wave of its workgroup loads, and
    some have none: each wave's report of them counts, those before the workgroup's first barrier too."""
    rng = np.random.default_rng(n)
    y0 = np.zeros((m, n), np.float32)
    y0[np.arange(m), np.where(np.arange(m) % 2 == 0, n - 1, 0)] = 1.0
    y0[rng.choice(m, size=m // 10, replace=False)] = 0.0
    layers = [offset_layer(rng, n, -0.01) for _ in range(2)]
    log(f"LDS widths, nonzero inputs: n={n} m={m}")
    run(n, layers, y0)


@pytest.mark.parametrize("nl", [4095, 4096])
def test_depth_of_the_read_back(nl):
    """Live counts of networks that the host's words hold and of deeper ones."""
    n, m = 32, 7
    rng = np.random.default_rng(nl)
    few = [offset_layer(rng, n, -0.01) for _ in range(3)]
    y0 = rng.random((m, n)).astype(np.float32)
    y0[2] = 0.0
    layers = [few[l % 3] for l in range(nl)]
    gpu = GpuNet(n, nl)
    ri = few[0][1]
    for l0 in range(0, nl, 512):
        part = layers[l0:l0 + 512]
        gpu.load(l0, np.stack([p[0] + i * ri.size for i, p in enumerate(part)]), np.concatenate([p[1] for p in part]),
                 np.concatenate([p[2] for p in part]), np.stack([p[3] for p in part]))
    log(f"{nl} layers")
    cats = gpu.run(y0)
    assert_parity(gpu, oracle_run(y0, layers), cats)


@pytest.mark.parametrize("n,m,scale", [(1024, 300, 1.0), (1024, 1, 1.0), (1000, 5000, 1.0), (6000, 700, 0.9), (6000, 60, 1.0)])
def test_final_rows_in_any_order(n, m, scale):
    """Final activations for ids that are unsorted, repeated, dead and alive, the whole list of categories, one
    run of it and none; categories and counts of more and fewer rows than one read-back word holds.
    Widths in LDS, rows by position (6000 neurons, 700 rows) and tiles (60 rows)."""
    rng = np.random.default_rng(n + m)
    dens = rng.uniform(0.3, 0.9, size=(m, 1)) if m > 1 else np.ones((1, 1))
    y0 = ((rng.random((m, n)) < dens) * np.float32(scale)).astype(np.float32)
    layers = [offset_layer(rng, n, -0.9) for _ in range(3)]
    gpu, cats = run(n, layers, y0)
    o = oracle_run(y0, layers)
    assert cats.size
    alive = np.zeros(m, bool)
    alive[cats] = True
    asked = [cats, cats[::-1], cats[:2], cats[1:1 + cats.size // 2], np.repeat(cats[:3], 2), rng.integers(0, m, size=50),
             np.empty(0, np.int64), np.arange(m)]
    if cats.size > 3:
        asked.append(np.r_[cats[0], cats[0], cats[2:cats.size]])
    for ids in asked:
        got = gpu.net.final_rows(ids)
        want = np.zeros((ids.size, n), np.float32)
        want[alive[ids]] = o.rows(ids[alive[ids]])
        np.testing.assert_array_equal(got, want)
    np.testing.assert_array_equal(gpu.net.categories(), cats)
    np.testing.assert_array_equal(gpu.net.live_counts(), oracle.padded_live_counts(o, 3))


@pytest.mark.parametrize("left", [1.5, 0.5])
def test_little_device_memory(left):
    """Layers whose segment streams don't fit the device's memory beside their lists, or whose lists need the memory
    of earlier layers' streams, load all the same; the network runs on tiles."""
    from tests.gpu_util import torch_cuda
    torch = torch_cuda()
    n, m, first, last = 16384, 300, 30, 40
    rng = np.random.default_rng(12)
    layers = []
    for i in range(2):
        cols = [np.sort(rng.choice(n, size=33, replace=False)) for _ in range(n)]
        cp, ri, v = csc(rng, n, cols, 0.125)
        layers.append((cp, ri, v, rng.uniform(-0.45, -0.35, size=n).astype(np.float32)))
    y0 = rng.random((m, n)).astype(np.float32)
    gpu = GpuNet(n, first + last)

    def many(layer, k):
        cp, ri, v, b = layer
        return np.stack([cp + i * ri.size for i in range(k)]), np.tile(ri, k), np.tile(v, k), np.tile(b, (k, 1))

    gpu.load(0, *many(layers[0], first))
    yd = torch.from_numpy(y0).cuda()
    nb = gpu.net.workspace_bytes(m)
    ws = torch.empty(nb, dtype=torch.uint8, device="cuda")
    lists = last * n * (33 * 8 + 4)  # what the lists and biases take; the streams take about as much
    torch.cuda.synchronize()
    log(f"little device memory, {left} of the lists")
    gc.collect()  # networks and tensors of earlier tests, and what torch keeps of them
    torch.cuda.empty_cache()
    fill, leave = [], int(left * lists)
    for _ in range(8):  # (the first reports of free memory are low, and torch may serve a piece from its own)
        more = torch.cuda.mem_get_info()[0] - leave
        if more > 32 << 20:
            fill.append(torch.empty(more, dtype=torch.uint8, device="cuda"))
    free = torch.cuda.mem_get_info()[0]
    if not leave - (8 << 20) < free < leave + (40 << 20):
        del fill
        torch.cuda.empty_cache()
        pytest.skip(f"{free >> 20} MiB are free where {leave >> 20} were to be left")
    try:
        gpu.load(first, *many(layers[1], last))
    finally:
        del fill
        torch.cuda.empty_cache()
    gpu.net.infer(yd, m, ws, nb, torch.cuda.current_stream())
    cats = gpu.net.categories()
    assert_parity(gpu, oracle_run(y0, [layers[0]] * first + [layers[1]] * last), cats)
    names = gpu.net.layer_kernels()
    assert names[1:] == ["k_layer_gfm"] * (first + last - 1) and cats.size
