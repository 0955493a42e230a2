"""Sizes at which the library's own choice of a launch changes: the longest list of a shape below the line and the shortest
one above it leave the same bytes as single wavefronts over the named list, which the parity tests compare with the oracle; and
lists of either kind that go out in several launches, against the oracle."""
import os
import re

import numpy as np
import pytest
import torch

from paper_2409_19256_amd import Plan, binding as B

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

# hidden, heads, head dim, ffn, vocab; train (p, t, d), generation (p_g, t_g).  Layers are added until a list is beyond the line.
SHAPES = {
    "whole_lines": ((512, 8, 64, 1408, 512), (1, 2, 1), (1, 1)),
    "rows_of_260_bytes": ((260, 4, 65, 896, 548), (1, 2, 1), (1, 1)),
    "rows_of_14_bytes": ((140, 4, 35, 28, 64), (1, 4, 1), (1, 2)),  # below a slot
    "three_destinations": ((256, 4, 64, 704, 512), (1, 4, 1), (1, 1)),
    "three_destinations_joined": ((384, 4, 96, 1324, 512), (1, 4, 1), (1, 1)),
    "seven_destinations": ((256, 8, 32, 712, 512), (1, 8, 1), (1, 1)),
    "seven_destinations_joined": ((136, 8, 17, 712, 512), (1, 8, 1), (1, 1)),  # eight with own pieces
}
FLAGS = {"execute": B.HF_SKIP_OWN, "refresh": B.HF_COPY_OWN, "from_gen": B.HF_GATHER_FROM_GEN, "install": B.HF_SKIP_OWN, "back": B.HF_SKIP_OWN}


def _limit(name):
    """A line of the library's sources, in bytes read once and written."""
    source = ""
    for name_of_file in ("abi.hip", "planner.cpp"):
        with open(os.path.join(ROOT, "paper_2409_19256_amd", "csrc", name_of_file)) as f:
            source += f.read()
    return int(re.search(r"constexpr uint64_t %s = (\d+)ull << 20;" % name, source).group(1)) << 20


def _plan(shape, layers, op, extra=0):
    (h, heads, hd, ffn, vocab), train, gen = SHAPES[shape]
    model = dict(n_layers=layers, hidden=h, n_q_heads=heads, n_kv_heads=heads, head_dim=hd, ffn=ffn, vocab=vocab)
    return Plan(model, train, gen, flags=FLAGS[op] | extra)


def _size_and_limits(shape, layers, op):
    with _plan(shape, layers, op, B.HF_PLAN_HOST_ONLY) as plan:
        if op == "install":
            size = 2 * sum(d.n_blocks * d.rows * d.row_bytes for r in plan.mat_ranks for d in plan.own_view(r))
            shared = False
        else:
            moved, read = (f(B.HF_DIR_GEN_TO_TRAIN if op == "back" else B.HF_DIR_TRAIN_TO_GEN) for f in (plan.bytes_moved, plan.unique_src_bytes))
            size, shared = moved + read, op != "back" and plan.get_param(B.HF_PARAM_AUTOMATIC_LIST) > 0
        if shared:
            return size, [_limit("kShortAutoList") * (1 if moved < 5 * read else 2)]
        return size, [_limit("kShortList"), _limit("kCachedList")]


def _depths(shape, op, line):
    """Layers of the longest list up to the line and of the shortest one beyond it."""
    size = lambda layers: _size_and_limits(shape, layers, op)
    lo, hi = 1, 2
    while size(hi)[0] <= size(hi)[1][line]:
        lo, hi = hi, 2 * hi
    while hi - lo > 1:
        mid = (lo + hi) // 2
        lo, hi = (mid, hi) if size(mid)[0] <= size(mid)[1][line] else (lo, mid)
    return lo, hi


def _random(n, seed):
    gen = torch.Generator(device="cuda").manual_seed(seed)
    return torch.randint(-32768, 32768, (n,), generator=gen, dtype=torch.int16, device="cuda")


def _calls():
    for shape in SHAPES:
        for op in FLAGS:
            shared = op in ("execute", "from_gen") and "destinations" in shape or op == "refresh"
            for line in range(1 if shared else 2):
                yield pytest.param(shape, op, shared, line, id=f"{shape}-{op}-{('short', 'cached')[line]}")


@pytest.mark.gpu
@pytest.mark.parametrize("shape,op,shared,line", _calls())
def test_both_sides_of_a_line_move_the_same_bytes(shape, op, shared, line):
    for side, layers in enumerate(_depths(shape, op, line)):
        size, limits = _size_and_limits(shape, layers, op)
        print(f"[{shape} {op} {layers} layers, {size} bytes, line at {limits[line]}]", flush=True)
        assert (len(limits) == 1) == shared and (size > limits[line]) == bool(side)
        with _plan(shape, layers, op) as plan:
            a, b = _random(plan.train_bytes // 2, 1), _random(plan.gen_bytes // 2, 2)
            results = []
            for threads in (0, 64):  # 64: the list of the mode in force, one wavefront per KiB
                plan.set_param(B.HF_PARAM_WG_THREADS, threads)
                t, g = a.clone(), b.clone()
                call = plan.back if op == "back" else plan.install_own if op == "install" else plan.execute
                call(t.data_ptr(), g.data_ptr())
                torch.cuda.synchronize()
                results.append((t, g))
            assert torch.equal(results[0][0 if op != "back" else 1], a if op != "back" else b)  # the source
            assert not torch.equal(results[0][1 if op != "back" else 0], b if op != "back" else a)
            for x, y in zip(*results):
                assert torch.equal(x, y)


@pytest.mark.gpu
@pytest.mark.parametrize("shape,layers", [("rows_of_260_bytes", 6), ("rows_of_260_bytes", 7), ("three_destinations_joined", 1),
                                          ("three_destinations_joined", 2), ("three_destinations_joined", 3)])
def test_lists_in_several_launches_match_oracle(shape, layers):
    """At most 1024 workgroups of 256 lanes to a launch.  Records per launch, and in the last one: way out and way back of six layers of the first
    shape (256 lanes) 204, 124 and 1024, 586, of seven (single wavefronts) 102, 74 and 512, 330; the second shape's automatic list of
    512 lanes 256, 66, its way back 341, 69 (256 lanes, two layers) and 170, 87 (single wavefronts, three): counts that are no
    multiples of the eight records that go to the eight XCDs together."""
    from oracle.reshard_oracle import GenLayout, Model, ReshardOracle, TrainLayout
    from paper_2409_19256_amd.arena import Arena
    from tests.oracle_util import POISON, seeded_train_buf

    (h, heads, hd, ffn, vocab), train_layout, gen_layout = SHAPES[shape]
    orc = ReshardOracle(Model(layers, h, heads, heads, hd, ffn, vocab), TrainLayout(*train_layout), GenLayout(*gen_layout))
    ranks = list(range(orc.n_ranks))
    train = seeded_train_buf(orc, 60 + layers)
    want = orc.reshard(train, np.full(orc.gen_region_offsets(ranks)[-1], POISON, np.uint16), ranks)
    back = orc.reshard_back(want, ranks, np.full(train.shape, POISON, np.uint16))
    tags, owner = orc.owner_tags(ranks), np.empty(want.shape, np.int32)
    for r, lo, hi in zip(ranks, orc.gen_region_offsets(ranks), orc.gen_region_offsets(ranks)[1:]):
        owner[lo:hi] = r
    own = tags == owner
    for op, line, side in {("rows_of_260_bytes", 6): [("execute", 0, 0), ("install", 0, 0), ("back", 0, 0)],
                           ("rows_of_260_bytes", 7): [("execute", 0, 1), ("install", 0, 1), ("back", 0, 1)],
                           ("three_destinations_joined", 1): [("execute", 0, 0)],
                           ("three_destinations_joined", 2): [("execute", 0, 1), ("install", 0, 0), ("back", 0, 0)],
                           ("three_destinations_joined", 3): [("install", 0, 1), ("back", 0, 1)]}[shape, layers]:
        size, limits = _size_and_limits(shape, layers, op)
        assert (size > limits[line]) == bool(side) and (line or size <= 192 << 20)
        assert size > 16 << 20  # more than 1024 workgroups of 8 KiB, read and written; less where the list is shared
        print(f"[several launches {shape} {layers} layers {op}]", flush=True)
        with _plan(shape, layers, op) as plan:
            plan.set_param(B.HF_PARAM_MAX_WGS_PER_LAUNCH, 1024)
            ar = Arena(plan)
            if op == "back":
                ar.gen.copy_(torch.from_numpy(want.view(np.int16)))
                ar.train.fill_(POISON - 0x10000)
                ar.back()
                result, expected = ar.train, back
            else:
                ar.train.copy_(torch.from_numpy(train.view(np.int16)))
                ar.gen.fill_(POISON - 0x10000)
                (ar.install_own if op == "install" else ar.execute)()
                result, expected = ar.gen, np.where(own == (op == "install"), want, POISON).astype(np.uint16)
            torch.cuda.synchronize()
            assert np.array_equal(result.cpu().numpy().view(np.uint16), expected)
