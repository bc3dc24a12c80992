"""The line between the two attention kernels for causal calls of short rows with more row groups than compute units: the
second work-group that a unit would get there is as long as the first, so the kernel of a work-group per row group loses.
Such a call does no more work than the same call without causality, which always takes the other kernel beyond a group per
unit, and must not take longer (it took 1.2 to 1.4 times as long on the wrong side of the line)."""
import pytest

pytestmark = pytest.mark.gpu


def graph_of(fn, launches):
    import torch
    side, graph = torch.cuda.Stream(), torch.cuda.CUDAGraph()
    with torch.cuda.stream(side):
        fn()
        side.synchronize()
        with torch.cuda.graph(graph, stream=side):
            for _ in range(launches):
                fn()
    return graph


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("N", [64, 128])
def test_short_causal_rows_do_not_take_longer_than_full_ones(N, d):
    import torch
    import paper_2502_18137_amd as sp
    units = torch.cuda.get_device_properties(0).multi_processor_count
    pairs = 2 * units // (N // 32)                      # two row groups per compute unit
    H = min(pairs, 128)
    g = torch.Generator(device="cuda").manual_seed(N)
    Q, K, V = (torch.randn(pairs // H, H, N, d, generator=g, device="cuda").to(torch.bfloat16) for _ in range(3))
    Qq, Kq, qs, ks, _ = sp.sparge_quantize(Q, K)
    tiles = sp.sparge_v_tiles(V)
    ws, outs, graphs = torch.empty(4096, dtype=torch.uint8, device="cuda"), [], []
    for causal in (False, True):
        outs.append(torch.empty_like(V))
        graphs.append(graph_of(lambda: sp.sparge_attn_tiled(Qq, Kq, qs, ks, tiles, V, None, -6.0, causal=causal, out=outs[-1], ws=ws), 50))
    times = [[], []]
    for _ in range(9):
        for k, graph in enumerate(graphs):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            graph.replay()
            b.record()
            torch.cuda.synchronize()
            times[k].append(a.elapsed_time(b) * 20)     # us a launch
    full, causal = (sorted(t)[len(t) // 2] for t in times)
    print(f"N={N} d={d}: {full:.2f} us, causal {causal:.2f}", flush=True)
    assert causal <= 1.12 * full
