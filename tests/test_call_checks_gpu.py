"""The binding's checks on GPU tensors: a call whose arguments are all as they
should be takes a short path, and anything else still meets the full checks."""
import pytest

pytestmark = pytest.mark.gpu


def _args(N=100, M=4, V=9, K=20):
    import torch
    g = torch.Generator(device="cuda")
    g.manual_seed(1)
    return dict(theta=torch.rand(M, K, device="cuda", generator=g),
                phi=torch.rand(V, K, device="cuda", generator=g),
                doc_id=(torch.arange(N, device="cuda") * M // N).int(),
                word_id=torch.randint(0, V, (N,), device="cuda", generator=g, dtype=torch.int32),
                u=torch.rand(N, device="cuda", generator=g))


BAD = {
    "theta": [lambda t: t.double(), lambda t: t[:, :19], lambda t: t.t(), lambda t: t.cpu(),
              lambda t: t[0], lambda t: None],
    "phi": [lambda t: t.half(), lambda t: t[:, :19].contiguous(), lambda t: t.cpu()],
    "doc_id": [lambda t: t.long(), lambda t: t[:50], lambda t: t[None], lambda t: t.cpu()],
    "word_id": [lambda t: t.float(), lambda t: t[::2], lambda t: t.cpu(), lambda t: [1, 2]],
    "u": [lambda t: t.double(), lambda t: t[:99], lambda t: t.cpu()],
    "out": [lambda t: t.long(), lambda t: t[:99], lambda t: t.cpu(), lambda t: t[None]],
}


@pytest.mark.parametrize("name", BAD)
def test_wrong_arguments_raise(name):
    import torch
    import paper_1505_03851_amd as lda
    for bad in BAD[name]:
        a = dict(_args(), out=torch.empty(100, dtype=torch.int32, device="cuda"))
        a[name] = bad(a[name])
        with pytest.raises((TypeError, ValueError)):
            lda.draw_butterfly(**a)
        if name not in ("u", "doc_id"):
            b = {k: v for k, v in a.items() if k not in ("u", "doc_id")}
            off = torch.tensor([0, 25, 50, 75, 100], device="cuda")
            with pytest.raises((TypeError, ValueError)):
                lda.draw_docs(b["theta"], b["phi"], off, b["word_id"], a["u"], out=b["out"])
            with pytest.raises((TypeError, ValueError)):
                lda.draw_philox(b["theta"], b["phi"], a["doc_id"], b["word_id"], 5, out=b["out"])


def test_status_codes_streams_and_outputs():
    import torch
    import paper_1505_03851_amd as lda
    a = _args()
    want = lda.draw_naive(**a)
    out = torch.full((100,), -1, dtype=torch.int32, device="cuda")
    side = torch.cuda.Stream()
    torch.cuda.synchronize()
    assert lda.draw_butterfly(**a, out=out, stream=side) is out
    side.synchronize()
    assert torch.equal(out, want)
    with torch.cuda.stream(side):
        got = lda.draw_butterfly(**a)
    side.synchronize()
    assert torch.equal(got, want) and got.dtype == torch.int32
    wide = dict(a, theta=torch.rand(4, 5000, device="cuda"), phi=torch.rand(9, 5000, device="cuda"))
    with pytest.raises(lda.LdaError) as e:  # K past the library's limit
        lda.draw_butterfly(**wide)
    assert e.value.status == lda.STATUS["LDA_ERR_UNSUPPORTED"]
    with pytest.raises(ValueError):
        lda.draw_butterfly(**dict(a, word_id=torch.full_like(a["word_id"], 9)), validate=True)
