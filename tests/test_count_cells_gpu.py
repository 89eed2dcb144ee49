"""The word counts by partition of the cells: calls of 524,288 tokens and more
whose document table can hold the partition, in the three forms, at the edges
of the chunks and of that rule, with one cell holding every token, with more
distinct cells than a bucket's table has slots (tokens counted in memory), with
tokens out of range, and into tables off their 16-byte boundary.  Integers:
every cell equals numpy's bincount."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu

MIN_N = 524288
CASES = [
    # (N, M, V, K, kind)
    (MIN_N - 1, 3000, 5000, 256, "zipf"),
    (MIN_N, 3000, 5000, 256, "zipf"),
    (MIN_N + 4095, 40000, 5000, 17, "zipf"),
    (MIN_N + 1, 600, 1000, 1000, "hot"),
    (MIN_N + 77, 2000, 40000, 333, "flat"),       # nearly every cell its own
    (MIN_N, 2100, 500, 256, "bad"),
    (MIN_N, 2113, 500, 257, "zipf"),              # the scratch just fits
    (MIN_N, 2064, 500, 256, "zipf"),              # ... and just does not
    (7999999, 70000, 30000, 128, "zipf"),
    (8000000, 70000, 30000, 128, "zipf"),
    (8000000 + 8191, 70000, 50000, 512, "flat"),  # tables overflow
    (6000001, 40000, 60000, 400, "flat"),         # ... the fewer ones of shorter calls
]


@pytest.mark.parametrize("N,M,V,K,kind", CASES)
def test_counts_by_partition(N, M, V, K, kind):
    import torch
    import paper_1505_03851_amd as lda
    g = np.random.Generator(np.random.PCG64(N + K))
    d = (np.arange(N, dtype=np.int64) * M // N).astype(np.int32)
    if kind == "hot":
        w = np.full(N, V - 1, np.int32)
        z = np.full(N, K - 1, np.int32)
    elif kind == "flat":
        w = g.integers(0, V, N, dtype=np.int32)
        z = g.integers(0, K, N, dtype=np.int32)
    else:
        w = (V * g.random(N) ** 6).astype(np.int32)
        z = (K * g.random(N) ** 3).astype(np.int32)
    if kind == "bad":
        w[::7], w[1::7], z[::5], z[2::5] = V, -1, K, -3
    want = oracle.counts(d, w, z, M, V, K)
    off = torch.from_numpy(np.searchsorted(d, np.arange(M + 1)).astype(np.int64)).cuda()
    td, tw, tz = (torch.from_numpy(a).cuda() for a in (d, w, z))
    p = torch.from_numpy(g.permutation(N)).cuda()

    def table(rows, shift):
        return torch.full((rows * K + shift,), -9, dtype=torch.int32,
                          device="cuda")[shift:].view(rows, K)

    index = lda.word_index_build(tw, V)
    for shift in (0, 1):
        print(f"[case] N={N} M={M} V={V} K={K} {kind} shift={shift}", flush=True)
        for name, got in (
                ("ids", lda.count_topics(td, tw, tz, M, V, K, table(M, shift), table(V, shift))),
                ("ids shuffled", lda.count_topics(td[p], tw[p], tz[p], M, V, K, table(M, shift),
                                                  table(V, shift))),
                ("offsets", lda.count_topics_docs(off, tw, tz, V, K, table(M, shift),
                                                  table(V, shift))),
                ("indexed", lda.count_topics_indexed(off, tw, tz, index, K, table(M, shift),
                                                     table(V, shift)))):
            for t, ref, what in zip(got, want, ("ndk", "nwk")):
                assert np.array_equal(t.cpu().numpy(), ref), (name, what)


def test_counts_by_partition_in_a_graph():
    """The call captured once and replayed on other topics, eager work between:
    each replay equals the eager call."""
    import torch
    import paper_1505_03851_amd as lda
    N, M, V, K = MIN_N + 100, 5000, 3000, 200
    gen = torch.Generator(device="cuda")
    gen.manual_seed(3)
    d = (torch.arange(N, device="cuda") * M // N).int()
    w = torch.randint(0, V, (N,), device="cuda", generator=gen, dtype=torch.int32)
    z = torch.zeros(N, device="cuda", dtype=torch.int32)
    ndk = torch.empty((M, K), dtype=torch.int32, device="cuda")
    nwk = torch.empty((V, K), dtype=torch.int32, device="cuda")
    s = torch.cuda.Stream()
    lda.count_topics(d, w, z, M, V, K, ndk, nwk)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=s):
        lda.count_topics(d, w, z, M, V, K, ndk, nwk)
    for rep in range(3):
        z.copy_(torch.randint(0, K, (N,), device="cuda", generator=gen, dtype=torch.int32))
        graph.replay()
        torch.cuda.synchronize()
        eager = lda.count_topics(d, w, z, M, V, K)
        torch.cuda.synchronize()
        assert torch.equal(ndk, eager[0]) and torch.equal(nwk, eager[1]), rep
        assert int(nwk.sum()) == N
