"""Decode attention of small batches, divided without a plan: every (request, kv
head) pair goes to one workgroup, to a fixed number of them, or is cut into
units whose size comes from the lengths; where the lengths are bad for that, the
call takes wave slices. At the edges of those divisions (no tokens, one tile,
chunks of 16 blocks and their remainders, fewer chunks than workgroups, more
chunks than workgroups, partials of more workgroups than a wavefront has lanes,
lengths far below the table's width, batches whose requests are taken longest
first, lengths just inside and far outside of what suits the division), for
every query group, against the oracle, across launch schedules and entry points,
and call after call on one workspace."""
import ctypes

import numpy as np
import pytest

import oracle
import paper_2411_01142_amd as neo
from paper_2411_01142_amd import workloads as W

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

# As for the planned kernels: weights as bf16 hi + lo are 2^-17 off at most, and
# a row's largest entry is smaller than the V entries it averages by up to
# sqrt(L); bounded by the row's largest entry times 2^-14.
REL_TOL = 2.0 ** -14


@pytest.fixture(scope="module", autouse=True)
def gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    neo.load_library()
    yield


CASES = {
    # name: (kv heads, lengths, extra table columns)
    "one_tile": (2, [1, 16, 2, 15], 0),
    "none": (4, [0, 0, 5, 0], 0),
    "one_part": (8, [512, 511, 497, 130, 128, 127, 0, 33], 0),
    "chunk_edges": (8, [255, 256, 257, 272, 528, 1, 0], 3),
    "fewer_chunks_than_parts": (1, [600, 40, 17, 3000, 0, 256], 0),
    "more_chunks_than_parts": (2, [70000, 300], 0),
    "one_long_many_short": (1, [30000] + [200] * 20 + [0, 1], 0),
    "wide_table": (8, [100, 900, 1, 300], 700),
    "most_pairs": (8, [1, 700, 333, 0] * 16 + [2048] * 64, 0),
    # more pairs than compute units: longest first
    "ordered": (4, [16 * (i * 37 % 200) + i % 17 for i in range(100)], 0),
    "ordered_equal": (8, [530] * 33, 0),
    "ordered_one_long": (2, [90] * 150 + [4000] + [0] * 20, 0),
    "ordered_rounds": (8, [(i * 353) % 2049 for i in range(180)], 0),
    "ordered_many_groups": (1, [(i * 7919) % 1000 for i in range(1000)], 1),
    # a pair's partials from more than 64 workgroups
    "pairs_196_workgroups": (1, [50021], 0),
    "pairs_128_workgroups": (2, [40000], 0),
    # units
    "units_of_16_blocks": (8, [1, 16, 0, 500, 512, 513, 528, 900, 17, 0, 40, 0], 300),
    "units_one_long": (1, [30000] + [200] * 40 + [0, 1, 512, 513], 0),
    "units_two_long": (1, [50021, 40000, 5], 0),
    "units_65_to_128_requests": (1, [(i * 353) % 2049 for i in range(128)], 100),
    "units_three_heads": (3, [(i * 977) % 3000 for i in range(40)], 0),
    "units_none": (8, [0] * 12, 200),
    "units_bad": (1, [6400] * 86, 0),
    # one workgroup a pair, in one round and in two
    "whole": (8, [(i * 353) % 1700 + 300 for i in range(30)] + [0, 1], 0),
    "whole_more_slices_than_pairs": (5, [1000 + 16 * i for i in range(30)], 0),
    "whole_bad": (8, [4096] + [150] * 29, 0),
    "whole_rounds": (8, [(i * 353) % 1537 + 512 for i in range(62)] + [0, 0], 200),
    "whole_rounds_512": (1, [(i * 353) % 3840 + 256 for i in range(510)] + [0, 1], 0),
    "whole_rounds_short": (4, [(i * 37) % 500 for i in range(100)], 50),
    "whole_rounds_bad": (8, [4096] + [150] * 61 + [0, 1], 0),
    "whole_rounds_halves": (8, [2048] * 33, 0),
    "whole_rounds_none": (8, [0] * 40, 60),
    "whole_three_rounds": (8, [(i * 353) % 1537 + 256 for i in range(94)] + [0, 1], 30),
    "whole_three_rounds_128": (6, [(i * 353) % 900 + 100 for i in range(128)], 0),
    "whole_three_rounds_short": (8, [(i * 37) % 200 for i in range(90)], 60),
    "whole_three_rounds_bad": (8, [4096] + [150] * 80, 0),
    "whole_three_rounds_thirds": (8, [512] * 65, 20),
    "pairs_three_rounds": (8, [(i * 37) % 513 for i in range(96)], 0),
    "pairs_768": (1, [(i * 37) % 500 for i in range(768)], 0),
}


@pytest.mark.parametrize("group", [1, 2, 4, 8, 16])
@pytest.mark.parametrize("name", list(CASES))
def test_pair_kernel_matches_the_oracle(name, group):
    hkv, lens, extra = CASES[name]
    case = W.build_case(lens, hkv * group, hkv, 128, 16, seed=7 * group + len(lens),
                        extra_table_cols=extra)
    print(f"[pairs] {name} G={group} Hkv={hkv} B={case.batch} mbps={case.max_blocks_per_seq}",
          flush=True)
    want = name.split("_")[0]
    if want in ("pairs", "units", "whole"):
        assert neo.debug_division(case.batch, case.num_q_heads, case.num_kv_heads,
                                  case.max_blocks_per_seq) == want
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
    assert np.array_equal(a, call())                     # counters are back at zero
    assert np.array_equal(a, call(schedule="two_kernel"))
    assert np.array_equal(a, call(schedule="staged"))
    # planned calls on the same workspace, before and after
    assert np.abs(call(max_slices=64) - a).max() <= 1e-5 * max(1.0, np.abs(a).max())
    assert np.array_equal(a, call())
    out = torch.full((case.batch, case.num_q_heads, 128), float("nan"), device="cuda")
    lib = neo.load_library()
    rc = lib.neo_decode_attention_noalloc(
        q.data_ptr(), k.data_ptr(), v.data_ptr(), bt.data_ptr(), sl.data_ptr(), case.num_q_heads,
        case.num_kv_heads, 128, 16, float(case.scale), out.data_ptr(), case.batch,
        case.max_blocks_per_seq, case.num_blocks, k.stride(0),
        ctypes.c_void_p(torch.cuda.current_stream().cuda_stream))
    assert rc == 0
    torch.cuda.synchronize()
    assert np.array_equal(a, out.cpu().numpy())
