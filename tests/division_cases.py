"""A decode call of every division, shared by the tests of the entry points (GPU):
no method arithmetic, only shapes and lengths."""
import paper_2411_01142_amd as neo
from paper_2411_01142_amd import workloads as W

# One call of every division: (kv heads, query heads per kv head, lengths, spare
# table columns). Units and whole pairs also with lengths that make them take
# wave slices.
DIVISION_CASES = {
    "wave_slices": (4, 4, [(i * 353) % 3000 for i in range(131)], 0),
    "head_slices": (16, 2, [(i * 97) % 900 + 40 for i in range(131)], 0),
    "head_slices_short": (4, 2, [(i * 7) % 60 for i in range(530)], 60),
    "pairs": (2, 4, [20000], 0),
    "units": (8, 4, [(i * 353) % 1500 for i in range(13)], 200),
    "whole": (8, 2, [(i * 353) % 1537 + 512 for i in range(48)], 0),
    "whole_skewed": (8, 2, [4096] + [150] * 50, 0),
}


def division_case(name):
    hkv, group, lens, extra = DIVISION_CASES[name]
    case = W.build_case(lens, hkv * group, hkv, 128, 16, seed=len(lens), extra_table_cols=extra)
    assert name.startswith(neo.debug_division(case.batch, case.num_q_heads, case.num_kv_heads,
                                              case.max_blocks_per_seq))
    return case
