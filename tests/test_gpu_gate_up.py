"""The gated pair in one launch beyond four rows and for groups below 128, against the oracle's fp64 products, at the
tolerance of every linear test (gpu_helpers); H comes from FP32 sums, so only its own rounding is new."""
import numpy as np
import pytest

import gwq_synth as gs
from oracle import gwq_oracle as orc

pytestmark = pytest.mark.gpu


def _pair(seed, N, K, bits, group=128, ppm=(10000, 10000)):
    layers = []
    for i in range(2):
        rng = np.random.default_rng([seed, i])
        W = gs.weight(N, K, rng, planted_cols=2)
        layers.append(orc.pack(W, gs.score_from_weight(W, rng), bits, ppm[i], group))
    return layers, np.random.default_rng([seed, 2])


def _check(layers, rng, M, what):
    import paper_2411_00850_amd as gwq
    from gpu_helpers import assert_close, to_gpu, upload_packed
    X = gs.activations(M, layers[0].K, rng)
    H = gwq.linear_gate_up(upload_packed(layers[0]), upload_packed(layers[1]), to_gpu(X)).cpu().numpy()
    assert_close(H, orc.gate_up(orc.linear_f64(layers[0], X), orc.linear_f64(layers[1], X)), what)


@pytest.mark.parametrize("bits", [4, 3])
@pytest.mark.parametrize("M", [5, 6, 7, 8, 9, 13, 16])
@pytest.mark.parametrize("N,K", [(16, 128), (1, 512), (50, 1152), (333, 2048), (130, 4096), (40, 5120)])
def test_every_row_count(bits, M, N, K):
    """Ragged last tiles, one wave to eight per layer, rows too long for the kernels (the product path), and different
    numbers of outliers in gate and up."""
    layers, rng = _pair(N + K + bits, N, K, bits, ppm=(10000, 30000))
    _check(layers, rng, M, f"gate_up N={N} K={K} M={M} bits={bits}")


@pytest.mark.parametrize("bits", [4, 3])
@pytest.mark.parametrize("tiles", [1, 2, 3, 7])
def test_streaming_pairs_of_tiles(bits, tiles):
    """The streaming kernel with one to seven tiles of each layer per block, the last block cut short."""
    import paper_2411_00850_amd as gwq
    layers, rng = _pair(77 + bits, 16 * 16 + 5, 2048, bits, ppm=(0, 20000))
    gwq.tuning_set("decode_tiles", tiles)
    try:
        for M in (9, 16):
            _check(layers, rng, M, f"gate_up tiles={tiles} M={M} bits={bits}")
    finally:
        gwq.tuning_set("decode_tiles", 0)


@pytest.mark.parametrize("bits", [4, 3])
@pytest.mark.parametrize("M", [9, 16])
@pytest.mark.parametrize("tiles", [2, 3])
def test_streaming_pairs_of_long_rows(bits, M, tiles):
    """Rows of 4096 (eight waves, two sets of threads that add up the tiles in turn), two and three tiles of each layer per block,
    the last block cut short; the up layer's outliers, 6 % of its weights, overflow the staged window of every tile."""
    import paper_2411_00850_amd as gwq
    layers, rng = _pair(31 * tiles + bits, 16 * 7 + 5, 4096, bits, ppm=(10000, 60000))
    gwq.tuning_set("decode_tiles", tiles)
    try:
        _check(layers, rng, M, f"gate_up K=4096 tiles={tiles} M={M} bits={bits}")
        _check(layers[::-1], rng, M, f"up and gate exchanged, tiles={tiles} M={M} bits={bits}")
    finally:
        gwq.tuning_set("decode_tiles", 0)


@pytest.mark.parametrize("N,K,M,bits,one_launch", [(8192, 2304, 9, 3, True), (9196, 2304, 9, 3, False),
                                                   (4096, 4992, 5, 3, True), (4999, 4992, 5, 3, False), (6200, 4992, 5, 3, True)])
def test_one_launch_where_it_is_the_faster_way(N, K, M, bits, one_launch):
    """Both sides of the rules in launch_decode: tiles shared out as evenly as by two products or not, blocks of ten waves
    that leave CUs uneven or not.  Which way was taken shows in the error against 64 bits: one launch rounds H alone
    (2^-11 / sqrt(3) relative and less), two products round G and U to FP16 as well, so about sqrt(3) as much."""
    import paper_2411_00850_amd as gwq
    from gpu_helpers import to_gpu, upload_packed
    layers, rng = _pair(N + K, N, K, bits)
    X = gs.activations(M, K, rng)
    H = gwq.linear_gate_up(upload_packed(layers[0]), upload_packed(layers[1]), to_gpu(X)).cpu().numpy().astype(np.float64)
    ref = orc.gate_up(orc.linear_f64(layers[0], X), orc.linear_f64(layers[1], X))
    error = np.linalg.norm(H - ref) / np.linalg.norm(ref)
    assert error < 5e-4 and (error < 2.0 ** -11 / 3 ** 0.5) == one_launch, error


@pytest.mark.parametrize("N,K,M,group,one_launch", [
    (16384, 1152, 2, 32, True), (16400, 1152, 2, 32, False), (16400, 1152, 6, 32, False), (16400, 1664, 2, 64, True),
    (2048, 2176, 3, 16, True), (4096, 2176, 3, 16, True), (4112, 2176, 3, 16, False), (12288, 2176, 1, 32, True), (14352, 2176, 1, 32, False),
    (2048, 3200, 4, 32, False), (2064, 3200, 4, 32, True), (2064, 4224, 3, 64, True), (6176, 4224, 3, 64, False),
    (5000, 2176, 7, 64, True), (2048, 3200, 5, 64, False), (2064, 3200, 5, 64, True),
    (2048, 4224, 5, 64, False), (2064, 4224, 5, 64, True), (4112, 4224, 5, 64, False)])
def test_small_groups_one_launch_where_it_is_the_faster_way(N, K, M, group, one_launch):
    """Both sides of launch_decode's rules for groups below 128.  One launch rounds H alone, two products round G and U to FP16
    first: H is nearer to the fp64 products so rounded, and one launch is the more exact."""
    import types
    import torch
    import paper_2411_00850_amd as gwq
    from gpu_helpers import download_packed, to_gpu
    bits = 3 + K // 128 % 2
    gen = torch.Generator(device="cuda")
    gen.manual_seed(N + K)
    rng = np.random.default_rng(N + K)
    X = gs.activations(M, K, rng)
    D, products = [], []
    for _ in range(2):                                  # packed on the GPU: byte for byte as the oracle packs
        W = torch.randn((N, K), generator=gen, device="cuda").mul_(0.02).half()
        D.append(gwq.pack(W, torch.rand((N, K), generator=gen, device="cuda"), bits, 10000, group=group))
        P = types.SimpleNamespace(N=N, K=K, bits=bits, group=group, **download_packed(D[-1]))
        products.append(orc.linear_f64(P, X))
    H = gwq.linear_gate_up(*D, to_gpu(X)).cpu().numpy().astype(np.float64)
    exact = orc.gate_up(*products)
    twice = orc.gate_up(*(y.astype(np.float16) for y in products)).astype(np.float16)
    off = [np.linalg.norm(H - ref) / np.linalg.norm(exact) for ref in (exact.astype(np.float16), twice, exact)]
    assert (off[0] < off[1]) == one_launch and off[2] < 5e-4, off


@pytest.mark.parametrize("bits", [4, 3])
@pytest.mark.parametrize("group", [16, 32, 64])
@pytest.mark.parametrize("N,K", [(50, 1152), (130, 4096), (20, 128)])
def test_small_groups(bits, group, N, K):
    layers, rng = _pair(group + N + bits, N, K, bits, group)
    for M in (1, 2, 3, 4, 7):
        _check(layers, rng, M, f"gate_up group={group} N={N} K={K} M={M} bits={bits}")


@pytest.mark.parametrize("bits", [4, 3])
@pytest.mark.parametrize("group", [16, 64, 128])
@pytest.mark.parametrize("N,K", [(16, 128), (50, 1152), (333, 2048), (77, 2432), (2070, 4096), (2100, 4992), (4200, 2176),
                                 (50, 6272), (77, 8192)])
def test_two_sets_of_waves(bits, group, N, K):
    """Up to eight rows with one set of waves for gate and one for up, and the calls beside them: one wave a set to eight, half
    a block per CU to two, ragged last tiles, both layers' outlier counts, the up layer's beyond a set's staged window (6 %)."""
    layers, rng = _pair(group + N + K + bits, N, K, bits, group, ppm=(10000, 60000 if N < 100 else 10000))
    for M in (1, 2, 3, 4, 5, 6, 7, 8) if N * K < 1000000 else (1, 4, 5, 8)[bits - 3::2]:
        _check(layers, rng, M, f"gate_up group={group} N={N} K={K} M={M} bits={bits}")


@pytest.mark.parametrize("M,group", [(1, 128), (5, 32), (8, 64)])
def test_two_sets_replayed_from_a_graph(M, group):
    test_replayed_from_a_graph(M, group)


@pytest.mark.parametrize("M,group", [(4, 16), (8, 128), (16, 128)])
def test_replayed_from_a_graph(M, group):
    import torch
    import paper_2411_00850_amd as gwq
    from gpu_helpers import to_gpu, upload_packed
    layers, rng = _pair(9 * M, 200, 2048, 4, group)
    D = [upload_packed(P) for P in layers]
    X = to_gpu(gs.activations(M, 2048, rng))
    H = torch.empty((M, 200), dtype=torch.float16, device="cuda")
    call = gwq.prepare_linear_gate_up(D[0], D[1], X, H)
    call()
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        call()
    for trial in range(3):
        X.copy_(to_gpu(gs.activations(M, 2048, rng)))
        want = gwq.linear_gate_up(D[0], D[1], X)
        H.fill_(float("nan"))
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(H, want), trial
