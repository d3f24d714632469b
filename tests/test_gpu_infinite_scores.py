"""Decode attention where some tokens' scores are minus infinity (a key with an
infinite entry, as a program writes it to mask a token): they weigh nothing, and
the rest of the request is averaged as without them, also where a whole tile, a
wavefront's tiles or a workgroup's share of a request holds no other score. For
every way a call is divided, against the oracle."""
import numpy as np
import pytest

import oracle
import paper_2411_01142_amd as neo
from paper_2411_01142_amd import workloads as W

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

# Weights as bf16 hi + lo are 2^-17 off at most, and a row's largest entry is
# smaller than the V entries it averages by up to sqrt(L).
REL_TOL = 2.0 ** -14
ONE, MINUS_INF = W.to_bf16(np.array([1.0, -np.inf], np.float32))


@pytest.fixture(scope="module", autouse=True)
def gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    neo.load_library()
    yield


def _masked(L, kind):
    """Tokens of a request of L tokens whose scores are minus infinity."""
    t = np.arange(L)
    return {0: t < 48,                 # the first tiles
            1: (t // 16) % 2 == 0,     # every other tile
            2: t < L - 1,              # all but the last token
            3: (t // 256) % 3 != 1,    # whole runs of 16 blocks
            4: t > 0,                  # all but the first token
            5: t < 0}[kind]            # none


def _mask(case):
    """Head dim 0 of every query is 1 and that of a masked token's key minus infinity."""
    case.q[:, :, 0] = ONE
    for b, L in enumerate(case.seq_lens):
        t = np.flatnonzero(_masked(int(L), b % 6))
        t = t[t != L - 1] if len(t) == L else t  # (a request keeps one token)
        case.k_cache[case.block_table[b, t // 16], :, 0, t % 16, 0] = MINUS_INF
    return case


CASES = {
    # name: (kv heads, group, lengths, calls)
    "one_workgroup_a_pair": (8, 4, [300, 500, 512, 17, 400, 90] * 6, [{}]),
    "few_workgroups_a_pair": (2, 8, [3000, 5000, 4111, 2900, 700, 16], [{}]),
    "many_workgroups_a_pair": (1, 1, [60000, 50021], [{}]),
    "more_pairs_than_compute_units": (4, 2, [(i * 353) % 2040 + 1 for i in range(90)], [{}]),
    "wave_slices": (3, 2, [(i * 353) % 2040 + 1 for i in range(90)],
                    [dict(max_slices=1024), dict(max_slices=200), dict(max_slices=1024, variant="valu")]),
    "wave_slices_long": (1, 4, [30000, 20011, 17, 9000], [dict(max_slices=1024)]),
    "head_slices": (16, 1, [5000] + [(i * 97) % 180 + 1 for i in range(160)], [{}]),
}


@pytest.mark.parametrize("name", list(CASES))
def test_scores_of_minus_infinity_weigh_nothing(name):
    hkv, group, lens, calls = CASES[name]
    case = _mask(W.build_case(lens, hkv * group, hkv, 128, 16, seed=len(lens)))
    q, k, v, bt, sl = case.to_torch("cuda", kv_layout="interleaved")
    ref = oracle.decode_attention(case)
    assert np.all(np.isfinite(ref))
    for kw in calls:
        for schedule in ("fused", "two_kernel", "staged"):
            print(f"[minus infinity] {name} {kw} {schedule}", flush=True)
            out = neo.decode_attention(q, k, v, bt, sl, scale=case.scale, schedule=schedule, **kw)
            a = out.cpu().numpy()
            bad = np.argwhere(~np.isfinite(a).all(axis=2))
            assert len(bad) == 0, f"{len(bad)} rows not finite, first (request, head) {bad[0]}"
            err = np.abs(a.astype(np.float64) - ref).max(axis=2)
            assert np.all(err <= REL_TOL * np.abs(ref).max(axis=2))
