"""The leaf-group kernel's index arithmetic on the CPU: the kernel's own source
built for the host (tests/leaf_host), a wavefront's lanes run in turn, under the
address sanitizer.  Every global array has its exact size, of LDS only the
running wavefront's region is accessible and a table load must stay inside its
row, so an access out of range in any launch shape ends the run; the topics are
compared with the oracle's.  Both table builds, every launch shape."""
import dataclasses
import os
import shutil
import subprocess

import numpy as np
import pytest

from paper_1505_03851_amd.inputs import doc_offsets, make_random
from parity import compare

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CLANG = shutil.which("clang++", path="/opt/rocm/llvm/bin" + os.pathsep + os.environ["PATH"])


@pytest.fixture(scope="module")
def programs(tmp_path_factory):
    if CLANG is None:
        pytest.skip("no clang++")
    out = tmp_path_factory.mktemp("leaf_host")
    procs = {}
    for wide in (0, 1):
        exe = str(out / f"leaf_host{wide}")
        procs[exe] = subprocess.Popen(
            [CLANG, "-x", "c++", "-std=c++17", "-O1", "-g1", "-w", "-mllvm", "-unroll-threshold=0",
             "-Xarch_host", "-fsanitize=address", f"-DLDA_WIDE_TABLES={wide}",
             "-I", os.path.join(HERE, "leaf_host"),
             "-I", os.path.join(ROOT, "paper_1505_03851_amd", "csrc"),
             os.path.join(HERE, "leaf_host", "leaf_host.cpp"), "-o", exe])
    assert all(p.wait() == 0 for p in procs.values())
    return list(procs)


def shape_of(N, M, K):
    """(G, H, C, KEEP, TOK) of the dispatch (TOK: of calls of many tokens)."""
    if K > 256:
        return 64, 2, 4, 0, 64
    if K > 128:
        return 64, 1, 8, 0, 64
    if K > 64:
        return (32, 1, 8, 1, 64) if N >= 128 * M else (32, 1, 4, 0, 64)
    if K > 32:
        return 16, 1, 8, 1, 64
    return (8, 1, 8, 0, 64) if K > 16 else (4, 1, 4, 0, 64)


def shapes_of(K):
    if 64 < K <= 128:
        return (32, 1, 8, 1, 64), (32, 1, 4, 0, 64)
    full = shape_of(1, 1, K)
    return (full, full[:4] + (16,)) if full[0] == 64 else (full,)


def draw(program, c, shape, tmp, form="ids", offsets=None, spread=0, first=0, step=1):
    src, dst = str(tmp / "in"), str(tmp / "out")
    docs = c.doc_id
    if form == "docs":
        docs = doc_offsets(c.doc_id, c.M) if offsets is None else offsets
    with open(src, "wb") as f:
        f.write(np.array([c.N, c.M, c.V, c.K, int(form == "docs")], np.int64).tobytes())
        for a in (c.theta, c.phi, docs, c.word_id, c.u):
            f.write(np.ascontiguousarray(a).tobytes())
    run = subprocess.run([program, src, dst, *map(str, (*shape, spread, first, step))],
                         stderr=subprocess.PIPE, text=True,
                         env=dict(os.environ, ASAN_OPTIONS="detect_leaks=0"))
    assert run.returncode == 0, run.stderr[:3000]
    return np.fromfile(dst, np.int32)


KS = [4, 15, 16, 17, 32, 33, 50, 64, 65, 101, 112, 128, 129, 131, 208, 255, 256, 257, 448, 511, 512]


@pytest.mark.parametrize("K", KS)
def test_every_shape_in_bounds(K, programs, tmp_path):
    for N, M, order in ((64 * 5 + 1, 2, "sequential"), (64 * 5 + 63, 12, "ragged"),
                        (64 * 2, 60, "ragged"), (64 * 3 + 17, 40, "shuffled"), (64, 1, "single")):
        c = make_random(N, M, 37, K, seed=K, alpha=0.5, beta=0.5, doc_order=order)
        for program in programs:
            for shape in shapes_of(K):
                for form in ("ids",) if order == "shuffled" else ("ids", "docs"):
                    z = draw(program, c, shape, tmp_path, form)
                    rep = compare(c, z)
                    assert rep.hard == 0, (shape, form, order, rep.first_hard)


@pytest.mark.parametrize("K", [20, 28, 32, 52, 64, 112, 128, 250, 256])
def test_eight_topic_leaves_in_bounds(K, programs, tmp_path):
    G = 4 if K <= 32 else 8 if K <= 64 else 16 if K <= 128 else 32
    for N, M, order in ((64 * 3 + 5, 8, "ragged"), (64 * 2 + 17, 40, "shuffled")):
        c = make_random(N, M, 37, K, seed=K, alpha=0.5, beta=0.5, doc_order=order)
        rep = compare(c, draw(programs[0], c, (G, 2, 4, 0, 64), tmp_path))
        assert rep.hard == 0, rep.first_hard


@pytest.mark.parametrize("K,M", [(112, 40), (66, 900), (128, 40), (131, 300), (256, 300)])
def test_scattered_documents_in_bounds(K, M, programs, tmp_path):
    """Stretches drawn by document class: two whole ones, an incomplete one."""
    N = 2 * 8192 + 700
    c = make_random(N, M, 200, K, seed=K, alpha=0.5, beta=0.5, doc_order="shuffled")
    z = draw(programs[0], c, shape_of(N, M, K), tmp_path, spread=11)
    rep = compare(c, z)
    assert rep.hard == 0, rep.first_hard


@pytest.mark.parametrize("kind,share", [
    ("shuffled", (0.08, 0.2)), ("one token each", None), ("two tokens each", None),
    ("one token each, backwards", None), ("by word", None), ("a document of 20%", (0.08, 0.2)),
    ("a document of 60%", None), ("two documents of 15%", (0.08, 0.2))])
def test_which_tokens_are_drawn_by_document_class(kind, share, programs, tmp_path):
    """Only scattered documents: not short ones in order, whose theta rows have no
    other reader, nor tokens word by word, nor those most of which are one
    document's; and each class gets about an eighth of the tokens, whatever the
    largest documents' shares.  (Every workgroup is run on
    its own: it draws its own 128 tokens, or a class's of half the stretch.)"""
    N, K = 4096, 66  # one stretch, 32 workgroups
    g = np.random.Generator(np.random.PCG64(5))
    M = {"one token": N, "two tokens": N // 2}.get(" ".join(kind.split()[:2]), 7000)
    d = np.arange(N) * M // N
    if kind == "one token each, backwards":
        d = d[::-1]
    elif kind == "by word":  # ascending in each of 20 words
        d = np.sort(g.integers(0, M, (20, N // 20 + 1)), axis=1).ravel()[:N]
    elif not kind.startswith(("one", "two tokens")):
        d = g.permutation(d)
        r = g.random(N)
        if kind.startswith("a document"):
            d[r < int(kind.split()[3][:-1]) / 100] = 11
        elif kind.startswith("two documents"):
            d[r < 0.3] = 11
            d[r < 0.15] = 6000
    c = make_random(64, 1, 50, K, seed=1)
    c = dataclasses.replace(c, theta=np.tile(c.theta, (M, 1)), doc_id=d.astype(np.int32),
                            word_id=g.integers(0, 50, N, dtype=np.int32),
                            u=g.random(N, dtype=np.float32))
    drawn = [draw(programs[0], c, shape_of(N, M, K), tmp_path, spread=11, first=b, step=0) >= 0
             for b in range(N // 128)]
    if share is None:
        for b, got in enumerate(drawn):
            assert got[128 * b:128 * (b + 1)].all() and got.sum() == 128, b
    else:
        of = np.array([got.sum() for got in drawn if got.any()]) / N
        assert len(of) == 8 and of.min() > share[0] and of.max() < share[1], of


@pytest.mark.parametrize("K", [48, 112, 208, 300])
def test_a_large_ragged_corpus_in_bounds(K, programs, tmp_path):
    """Documents as offsets over six million tokens of lognormal lengths, empty
    documents among them: wavefronts of the whole range."""
    N, M = 6_000_001, 87_112
    g = np.random.Generator(np.random.PCG64(K))
    x = g.lognormal(0.0, 0.8, M) * (g.random(M) > 0.1)
    x[-3:] = 0
    off = np.concatenate([[0], np.rint(np.cumsum(x) * (N / x.sum()))]).astype(np.int64)
    off[-4:] = N
    ids = np.repeat(np.arange(M, dtype=np.int32), np.diff(off))
    c = make_random(64, 5, 97, K, seed=K, alpha=0.5, beta=0.5)
    c = dataclasses.replace(c, theta=np.tile(c.theta, (M // 5 + 1, 1))[:M], doc_id=ids,
                            word_id=g.integers(0, 97, N, dtype=np.int32),
                            u=g.random(N, dtype=np.float32))
    z = draw(programs[0], c, shape_of(N, M, K), tmp_path, "docs", off, first=3, step=2503)
    at = np.flatnonzero(z >= 0)
    assert at.size >= 18 * 128 and at[-1] == N - 1
    part = dataclasses.replace(c, doc_id=ids[at], word_id=c.word_id[at], u=c.u[at])
    rep = compare(part, z[at])
    assert rep.hard == 0, rep.first_hard


@pytest.mark.parametrize("K", [50, 112, 208])
def test_any_offsets_stay_in_bounds(K, programs, tmp_path):
    """Offsets that are no offsets (unordered, negative, past N): some document
    is drawn from, and nothing outside the arrays is touched."""
    N, M = 64 * 7 + 9, 30
    c = make_random(N, M, 37, K, seed=K, alpha=0.5, beta=0.5)
    g = np.random.Generator(np.random.PCG64(K))
    for kind in range(6):
        off = [np.full(M + 1, 2 ** 62), np.full(M + 1, -2 ** 62), np.full(M + 1, N),
               g.integers(-5 * N, 5 * N, M + 1), g.permutation(doc_offsets(c.doc_id, M)),
               np.arange(M, -1, -1) * (N // M)][kind].astype(np.int64)
        z = draw(programs[0], c, shape_of(N, M, K), tmp_path, "docs", off)
        assert z.min() >= 0 and z.max() < K


@pytest.mark.parametrize("K", [5, 12, 20, 50, 112, 131, 208, 300, 500])
def test_any_weights_and_uniforms_give_topics(K, programs, tmp_path):
    """Uniforms below 0, above 1 and NaN, weights below 0, infinite and NaN: the
    draw has no meaning, but it is a topic (one that indexes theta and phi)."""
    N, M = 64 * 4, 6
    c = make_random(N, M, 37, K, seed=K, alpha=0.5, beta=0.5)
    u, theta, phi = c.u.copy(), c.theta.copy(), c.phi.copy()
    u[::5], u[1::7], u[2::9], u[3::11] = -0.5, np.nan, 1.5, np.inf
    theta[1, ::3], theta[2, ::5], theta[3, K // 2], theta[4] = -theta[1, ::3], np.nan, np.inf, 0
    phi[::7, 0] = np.inf
    for kw in (dict(u=u), dict(theta=theta), dict(theta=-c.theta), dict(u=u, theta=theta, phi=phi)):
        bad = dataclasses.replace(c, **kw)
        for program in programs:
            for shape in shapes_of(K):
                z = draw(program, bad, shape, tmp_path)
                assert z.min() >= 0 and z.max() < K


@pytest.mark.parametrize("M", [1, 100, 2 ** 30 + 12345, 1_900_000_000, 2 ** 31 - 1])
def test_document_search_among_very_many_documents(M, tmp_path):
    """Every token in the last of up to 2^31 - 1 documents: the search's steps
    double up to the number of documents and stay inside them."""
    if CLANG is None:
        pytest.skip("no clang++")
    exe = str(tmp_path / "doc_search")
    subprocess.run([CLANG, "-x", "c++", "-std=c++17", "-O1", "-w",
                    "-I", os.path.join(HERE, "leaf_host"),
                    "-I", os.path.join(ROOT, "paper_1505_03851_amd", "csrc"),
                    os.path.join(HERE, "leaf_host", "doc_search.cpp"), "-o", exe], check=True)
    N = 1 << 20
    at = [0, 64, N // 64, N // 16, N // 8, N // 5, N // 2, N - 64]
    run = subprocess.run([exe, str(M), str(N), *map(str, at)], stdout=subprocess.PIPE, text=True)
    assert run.returncode == 0, (run.returncode, run.stdout)
    assert run.stdout.split() == [str(M - 1)] * (2 * len(at))
