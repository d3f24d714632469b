"""The binding's one-pass tensor check against the full checks: over strides,
types, dims and devices, it accepts nothing that they refuse, gives the same
block stride, and what it does not accept is still accepted or refused by the
full checks."""
import itertools

import pytest

import paper_2411_01142_amd as neo
from paper_2411_01142_amd import workloads as W

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    neo.load_library()
    yield


def _forms(t):
    """t and tensors of its shape (or nearly) that differ in one respect."""
    out = [t, torch.nn.Parameter(t, requires_grad=False) if t.is_floating_point() else t.clone(),
           t.cpu(), t.to(torch.float16) if t.is_floating_point() else t.to(torch.int64),
           t.unsqueeze(0), t[0]]
    if t.dim() > 1:
        pad = torch.zeros((t.shape[0], *t.shape[1:-1], t.shape[-1] + 8), dtype=t.dtype,
                          device=t.device)
        out += [pad[..., :t.shape[-1]], t.transpose(-1, -2).contiguous().transpose(-1, -2),
                t[::2], t.repeat_interleave(2, 0)[::2]]
    else:
        out.append(t.repeat_interleave(2)[::2])
    return out


def _full(k, v, table, lens):
    try:
        stride = neo._shared_stride(k, "k", v, "v")
        neo._require(table, "table", torch.int32, 2)
        neo._require(lens, "lens", torch.int32, 1)
        return stride
    except (TypeError, ValueError):
        return None


@pytest.mark.parametrize("layout,pad", [("separate", 0), ("interleaved", 0), ("interleaved", 40)])
def test_one_pass_check_accepts_only_what_the_full_checks_accept(layout, pad):
    case = W.build_case([20, 40, 5, 1], 8, 2, 128, 16, seed=4)
    q, k, v, bt, sl = case.to_torch("cuda", kv_layout=layout, kv_pad=pad)
    full = _full(k, v, bt, sl)
    assert full == k.stride(0) and neo._paged_stride(torch, q.device, k, v, bt, sl) == full
    accepted = 0
    for a, b in itertools.combinations(range(4), 2):
        base = [k, v, bt, sl]
        for x, y in itertools.product(_forms(base[a]), _forms(base[b])):
            args = list(base)
            args[a], args[b] = x, y
            got = neo._paged_stride(torch, q.device, *args)
            assert got is None or got == _full(*args), (a, b, x.stride(), y.stride())
            accepted += got is not None
    assert accepted > 0
    assert neo._paged_stride(torch, torch.device("cpu"), k, v, bt, sl) is None
    assert neo._paged_stride(torch, None, None, v, bt, sl) is None


def test_forms_outside_the_one_pass_check_are_still_accepted():
    case = W.build_case([20, 40, 5, 1], 8, 2, 128, 16, seed=5)
    q, k, v, bt, sl = case.to_torch("cuda")
    want = neo.decode_attention(q, k, v, bt, sl)
    P = torch.nn.Parameter
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    got = neo.decode_attention(P(q, requires_grad=False), P(k, requires_grad=False), v, bt, sl,
                               stream=side)
    side.synchronize()
    assert torch.equal(got, want)
    with pytest.raises(TypeError):
        neo.decode_attention(q.float(), k, v, bt, sl)
    with pytest.raises(ValueError, match="on a GPU"):
        neo.decode_attention(q, k, v, bt.cpu(), sl)
    with pytest.raises(ValueError, match="contiguous"):
        neo.kv_append(k, v, q[:, :2].transpose(0, 1).contiguous().transpose(0, 1), q[:, :2], bt, sl)
