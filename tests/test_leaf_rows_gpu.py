"""The leaf-group kernel at the edges of its rows: K around every group width
(16, 32, 64, 128, 256, 512), K of every remainder mod 4 (the first quad of a
row then holds 1 to 3 topics), documents of every mode (one per group, a few
runs, any), the window's tail, and both table builds."""
import dataclasses

import numpy as np
import pytest

from paper_1505_03851_amd.inputs import make_random
from parity import compare, run_kernel, to_device

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("K", [4, 5, 15, 16, 17, 30, 33, 63, 65, 67, 126, 129, 131, 250, 255, 257,
                               259, 385, 447, 509, 511, 512])
def test_rows_of_every_width(K):
    # documents of 128 tokens (with 32-lane groups: sums kept in registers),
    # of about 20 (runs), one token each in turn (any)
    for N, M, order in ((64 * 33 + 1, 16, "sequential"), (64 * 33 + 63, 100, "ragged"),
                        (64 * 9 + 17, 40, "shuffled")):
        # (weights away from fp32's subnormal range, where products vanish)
        c = make_random(N, M, 300, K, seed=K, alpha=0.5, beta=0.5, doc_order=order)
        dev = to_device(c)
        z = {k: run_kernel(k, dev) for k in ("butterfly", "variant-wide", "variant-leaf8")}
        for name, got in z.items():
            rep = compare(c, got)
            print(f"[parity] {c.name} {name}: {rep}", flush=True)
            assert rep.hard == 0, (name, rep.first_hard)
        assert np.array_equal(z["butterfly"], z["variant-wide"])


@pytest.mark.parametrize("K", [130, 256, 257, 512])
@pytest.mark.parametrize("N", [64, 65, 79, 65536, 65537, 98304, 98305, 196609, 393153])
def test_few_and_many_tokens_per_wavefront(N, K):
    """64-lane groups at the edges of the rule that gives a wavefront 16 tokens,
    and of such a wavefront: every form of the documents."""
    for M, order in ((max(1, N // 128), "sequential"), (max(1, N // 30), "ragged"),
                     (50, "shuffled")):
        c = make_random(N, M, 300, K, seed=K, alpha=0.5, beta=0.5, doc_order=order)
        dev = to_device(c)
        for name in ("butterfly", "variant-wide") + (("docs",) if order != "shuffled" else ()):
            rep = compare(c, run_kernel(name, dev))
            assert rep.hard == 0, (name, order, rep.first_hard)


@pytest.mark.parametrize("K", [5, 18, 35, 66, 131, 259])
def test_tiny_uniforms_behind_empty_components(K):
    """Stops of 0 and of a few ulps of S, and the largest u, with every second
    topic weightless: no draw ends in an empty component of the first quad or
    at a topic the rounding band does not admit."""
    N = 640
    c = make_random(N, 8, 60, K, seed=K, alpha=0.5, beta=0.5)
    theta = c.theta.copy()
    theta[1::2, ::2] = 0.0
    theta[0] = 0.0
    u = (np.arange(N) % 5).astype(np.float32) * np.float32(2.0 ** -24)
    u[4::5] = np.float32(1.0 - 2.0 ** -24)
    c = dataclasses.replace(c, theta=theta, u=u)
    for kernel in ("butterfly", "variant-wide"):
        rep = compare(c, run_kernel(kernel, to_device(c)))
        assert rep.hard == 0, (kernel, rep.first_hard)


@pytest.mark.parametrize("N,M,K", [((1 << 20), 16000, 128), ((1 << 20) + 4095, 24000, 101),
                                   ((1 << 20) + 77, 7000, 256), ((1 << 20) + 4096, 9000, 190),
                                   ((1 << 20) + 1, 30000, 66),
                                   # 40 tokens per document and more: listed by class; 128:
                                   # 32-lane groups that keep their sums, full and padded rows
                                   ((1 << 20) + 1, 25000, 66), (1 << 21, 16384, 128),
                                   (2200000, 17000, 101)])
@pytest.mark.parametrize("order", ["shuffled", "partly"])
def test_scattered_documents(N, M, K, order):
    """Tokens in no document order, with theta past an XCD's L2: stretches of
    the tokens are drawn by document class; "partly": stretches of either kind,
    and a last one that is incomplete."""
    c = make_random(N, M, 500, K, seed=K, alpha=0.5, beta=0.5,
                    doc_order="shuffled" if order == "shuffled" else "sequential")
    if order == "partly":
        g = np.random.Generator(np.random.PCG64(K))
        d = c.doc_id.copy()
        for lo, hi in ((5000, 300000), (N - 9000, N)):
            d[lo:hi] = g.permutation(d[lo:hi])
        c = dataclasses.replace(c, doc_id=d)
    dev = to_device(c)
    z = {k: run_kernel(k, dev) for k in ("butterfly", "variant-wide")}
    rep = compare(c, z["butterfly"])
    print(f"[parity] {c.name} {order}: {rep}", flush=True)
    assert rep.hard == 0, rep.first_hard
    assert np.array_equal(z["butterfly"], z["variant-wide"])
    import torch
    import paper_1505_03851_amd as lda
    a = (dev["theta"], dev["phi"], dev["doc_id"], dev["word_id"])
    zp = lda.draw_philox(*a, 7, 3)
    assert torch.equal(zp, lda.draw_butterfly(*a, lda.philox_uniforms(N, 7, 3)))
