"""Decode attention with one slice per workgroup over groups of four kv heads:
batches large enough to take that plan, at its edges (empty and one-token
requests, whole blocks, requests cut between many slices, more finished pairs
in a slice than its LDS holds, more requests in a slice than a wavefront has
lanes), and batches that take wave slices in its place because they are short,
for every query group, against the oracle and across launch schedules."""
import numpy as np
import pytest

import oracle
import paper_2411_01142_amd as neo
from paper_2411_01142_amd import workloads as W

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

# The softmax weights enter the second product as bf16 hi + lo, 2^-17 of each
# weight off at most; a row, a convex combination of V rows, is then off by
# 2^-17 of the largest V entries, and its own largest entry is smaller than
# those by up to sqrt(L): bounded here by the row's largest entry times 2^-14.
REL_TOL = 2.0 ** -14


@pytest.fixture(scope="module", autouse=True)
def gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    neo.load_library()
    yield


def _lens(kind, batch, rng):
    if kind == "short":     # many pairs a slice, several of one tile
        x = rng.integers(0, 40, batch)
        x[:3] = [1, 0, 700]  # (the table's width is part of the plan's rule)
    elif kind == "blocks":  # whole blocks only
        x = 16 * rng.integers(0, 60, batch)
    elif kind == "runs":    # runs of empty requests longer than a wavefront
        x = np.where(np.arange(batch) % 90 < 3, rng.integers(1200, 3000, batch), 0)
    elif kind == "ones":    # one block each: more than 64 requests in a slice
        x = rng.integers(1, 17, batch)
        x[5] = 600
    else:                   # a few requests over many slices, between short ones
        x = np.where(rng.random(batch) < 0.02, rng.integers(3000, 9000, batch),
                     rng.integers(1, 120, batch))
        x[0] = 5000
    return x


@pytest.mark.parametrize("group", [1, 2, 4, 8, 16])
@pytest.mark.parametrize("kind", ["short", "blocks", "long", "runs", "ones"])
def test_head_slices_match_the_oracle(group, kind):
    rng = np.random.default_rng(100 * group + len(kind))
    hkv = 16 if group <= 4 else 4
    batch = 2048 // hkv + 3  # more than two pairs of four heads per compute unit
    batch *= 4 if hkv == 4 else 1
    if kind in ("runs", "ones"):
        hkv, batch = 4, 18000 if kind == "ones" else 1800
    _check(group, hkv, _lens(kind, batch, rng), kind, extra=3)


@pytest.mark.parametrize("group", [1, 4, 16])
@pytest.mark.parametrize("positions", [6143, 6144])
def test_around_the_least_positions_of_head_slices(group, positions):
    # 24 positions per compute unit (a pair of n blocks has n + 1): one fewer
    # takes wave slices.
    lens = np.zeros(520, np.int64)
    lens[20:381] = 256                              # 17 positions each
    lens[510] = 16 * (positions - 361 * 17 - 1) - 3
    _check(group, 4, lens, f"{positions} positions", extra=40)


def _check(group, hkv, lens, kind, extra):
    case = W.build_case(lens.tolist(), hkv * group, hkv, 128, 16, seed=group,
                        extra_table_cols=extra)
    print(f"[heads] G={group} Hkv={hkv} B={case.batch} {kind} sumL={case.total_tokens()}", flush=True)
    assert neo.debug_division(case.batch, case.num_q_heads, hkv,
                              case.max_blocks_per_seq) == "head_slices"
    q, k, v, bt, sl = case.to_torch("cuda", kv_layout="interleaved")
    ws = neo.new_workspace(case.batch, case.num_q_heads, case.num_kv_heads)

    def call(**kw):
        out = torch.full((case.batch, case.num_q_heads, 128), float("nan"), device="cuda")
        neo.decode_attention(q, k, v, bt, sl, scale=case.scale, out=out, workspace=ws, **kw)
        torch.cuda.synchronize()
        return out.cpu().numpy()

    a = call()
    ref = oracle.decode_attention(case)
    err = np.abs(a.astype(np.float64) - ref).max(axis=2)
    assert np.all(np.isfinite(a))
    assert np.all(err <= REL_TOL * np.abs(ref).max(axis=2))
    assert np.array_equal(a, call())                          # counters are back at zero
    assert np.array_equal(a, call(schedule="two_kernel"))
    assert np.array_equal(a, call(schedule="staged"))
