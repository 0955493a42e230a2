"""The list that hf_reshard_execute runs while every choice is the library's (Plan::dev_auto): the records and
bands against the tile lists, byte by byte (host code, under AddressSanitizer and UndefinedBehaviorSanitizer), and the
kernel against the oracle at the edges of slots, lines, stripes and wavefronts."""
import os
import shutil
import subprocess

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.mark.skipif(shutil.which("g++") is None, reason="g++ not available")
def test_the_automatic_list_moves_the_bytes_of_the_tiles(tmp_path):
    exe = str(tmp_path / "auto_list")
    csrc = os.path.join(ROOT, "paper_2409_19256_amd", "csrc")
    subprocess.run(["g++", "-std=c++17", "-O2", "-g", "-fsanitize=address,undefined", "-fno-sanitize-recover=all", "-static-libasan",
                    "-I", os.path.join(ROOT, "include"), "-I", csrc, os.path.join(csrc, "planner.cpp"),
                    os.path.join(ROOT, "tests", "auto_list_main.cpp"), "-o", exe], check=True, capture_output=True, text=True)
    env = dict(os.environ, ASAN_OPTIONS="detect_leaks=1:abort_on_error=0:verify_asan_link_order=0")
    r = subprocess.run([exe], capture_output=True, text=True, env=env, timeout=300)
    assert r.returncode == 0 and r.stdout == "ok\n", r.stdout + r.stderr


def test_the_plan_says_which_list_runs():
    from paper_2409_19256_amd import binding as B
    from tests.cases import SMALL
    from tests.libcases import make_plan

    with make_plan(SMALL[0], B.HF_PLAN_HOST_ONLY, mat=[0, 2]) as pl:  # one rank per group: no piece has two destinations
        assert pl.get_param(B.HF_PARAM_AUTOMATIC_LIST) == 0
    with make_plan(SMALL[1], B.HF_PLAN_HOST_ONLY) as pl:
        records = pl.get_param(B.HF_PARAM_AUTOMATIC_LIST)
        assert records > 0
        with pytest.raises(B.HfError):
            pl.set_param(B.HF_PARAM_AUTOMATIC_LIST, 1)  # to be read only
        for param, named, automatic in [(B.HF_PARAM_MULTICAST, B.HF_MULTICAST_PREFETCHED, B.HF_MULTICAST_AUTO),
                                        (B.HF_PARAM_VARIANT, B.HF_VARIANT_LDS_STAGED, B.HF_VARIANT_PARTS), (B.HF_PARAM_WG_THREADS, 64, 0),
                                        (B.HF_PARAM_PART_BYTES, 1024, 0), (B.HF_PARAM_CACHE_POLICY, 1, -1)]:
            pl.set_param(param, named)
            assert pl.get_param(B.HF_PARAM_AUTOMATIC_LIST) == 0
            pl.set_param(param, automatic)
            assert pl.get_param(B.HF_PARAM_AUTOMATIC_LIST) == records


# stripes of 14 bytes (records), then of 16 to 2752 bytes: every length of a joined slot's first part, around a slot, a line and a KiB
COLS = [7, 8, 9, 10, 11, 12, 13, 14, 15, 16, 17, 63, 64, 65, 511, 513, 1376]
LAYOUTS = ["t4 own left out", "t4 whole", "t8 p2 merged", "t2 registers", "from gen"]
MIB = 1 << 20


# On either side of the size up to which eight wavefronts go to a workgroup, unpaced: 32 MiB, 64 from five destinations on.  Longer lists
# (a longer vocabulary) run single wavefronts, paced from three destinations on.
@pytest.mark.gpu
@pytest.mark.parametrize("layout,cols,side", [(layout, cols, side) for layout in LAYOUTS for cols in COLS for side in ("short", "long")
                                              if (layout, cols, side) != ("t8 p2 merged", 1376, "short")])  # long with any vocabulary
def test_automatic_list_matches_oracle(layout, cols, side):
    import torch

    from oracle.reshard_oracle import GenLayout, Model, ReshardOracle, TrainLayout
    from paper_2409_19256_amd import binding as B
    from paper_2409_19256_amd.arena import Arena
    from tests.libcases import make_plan
    from tests.oracle_util import POISON, seeded_train_buf

    p, t, tg, flags = {"t4 own left out": (1, 4, 1, 0), "t4 whole": (1, 4, 1, B.HF_COPY_OWN), "t8 p2 merged": (2, 8, 2, 0),
                       "t2 registers": (1, 2, 1, B.HF_COPY_OWN), "from gen": (1, 4, 1, B.HF_GATHER_FROM_GEN)}[layout]
    print(f"[auto cols {cols} {layout} {side}]", flush=True)
    vocab = t * (13 if side == "short" else {2: 21001, 4: 7509, 8: 3755}[t])
    case = dict(name="auto", model=Model(2 * p, 72, t, t, 9, t * cols, vocab), train=TrainLayout(p, t, 1), gen=GenLayout(1, tg))
    orc = ReshardOracle(case["model"], case["train"], case["gen"])
    ranks = list(range(orc.n_ranks))
    train = seeded_train_buf(orc, 700 + cols)
    want = orc.reshard(train, np.full(orc.gen_region_offsets(ranks)[-1], POISON, np.uint16), ranks)
    tags = orc.owner_tags(ranks)
    poison = POISON - 0x10000
    with make_plan(case, flags) as pl:
        assert pl.get_param(B.HF_PARAM_AUTOMATIC_LIST) > 0  # that is what runs
        moved, read = pl.bytes_moved(0), pl.unique_src_bytes(0)
        assert (moved + read <= (32 if moved < 5 * read else 64) * MIB) == (side == "short")
        ar = Arena(pl)
        ar.train.copy_(torch.from_numpy(train.view(np.int16)))
        start = want.copy()
        for i, r in enumerate(ranks):
            lo, hi = orc.gen_region_offsets(ranks)[i:i + 2]
            # what is gathered is poisoned; the own pieces hold other bytes than the training shard's, and stay
            # (gathered out of the generation buffers they are the source)
            start[lo:hi][(tags[lo:hi] >= 0) & (tags[lo:hi] != r)] = POISON
            if flags != B.HF_GATHER_FROM_GEN:
                start[lo:hi][tags[lo:hi] == r] = 0x1234
                if flags != B.HF_COPY_OWN:
                    want[lo:hi][tags[lo:hi] == r] = 0x1234
        ar.gen.copy_(torch.from_numpy(start.view(np.int16)))
        assert poison < 0
        for _ in range(2):
            ar.execute()
        torch.cuda.synchronize()
        assert np.array_equal(ar.gen.cpu().numpy().view(np.uint16), want)


@pytest.mark.gpu
@pytest.mark.parametrize("copy_own", [False, True], ids=["own left out", "whole"])
def test_automatic_list_in_several_launches(copy_own):
    """A list of more workgroups than one launch may have, cut between records of rows and of bands alike."""
    import torch

    from paper_2409_19256_amd import binding as B
    from paper_2409_19256_amd.arena import Arena
    from tests.cases import MEDIUM
    from tests.libcases import make_plan
    from tests.oracle_util import POISON, make_oracle, seeded_train_buf

    for case in MEDIUM[:2]:
        print(f"[several launches {case['name']}]", flush=True)
        orc = make_oracle(case)
        ranks = list(range(orc.n_ranks))
        train = seeded_train_buf(orc, 21)
        want = orc.reshard(train, np.full(orc.gen_region_offsets(ranks)[-1], POISON, np.uint16), ranks)
        tags = orc.owner_tags(ranks)
        with make_plan(case, B.HF_COPY_OWN if copy_own else 0) as pl:
            pl.set_param(B.HF_PARAM_MAX_WGS_PER_LAUNCH, 1024)  # 4096 workgroups of one wavefront, a KiB each
            assert pl.get_param(B.HF_PARAM_AUTOMATIC_LIST) > 0 and pl.unique_src_bytes(0) > 3 * 4096 * 1024
            ar = Arena(pl)
            ar.train.copy_(torch.from_numpy(train.view(np.int16)))
            start = np.full(want.shape, POISON, np.uint16)
            if not copy_own:
                for i, r in enumerate(ranks):
                    lo, hi = orc.gen_region_offsets(ranks)[i:i + 2]
                    start[lo:hi][tags[lo:hi] == r] = 0x1234
                    want[lo:hi][tags[lo:hi] == r] = 0x1234
            ar.gen.copy_(torch.from_numpy(start.view(np.int16)))
            ar.execute()
            torch.cuda.synchronize()
            assert np.array_equal(ar.gen.cpu().numpy().view(np.uint16), want)


@pytest.mark.gpu
def test_a_captured_graph_outlives_launch_parameters_that_name_another_list():
    """Each of the four launch parameters is taken away from the library's choice and given back: the call then runs another list, and a
    graph that holds the library's own still replays, before, between and after."""
    import torch

    from paper_2409_19256_amd import binding as B
    from paper_2409_19256_amd.arena import Arena
    from tests.cases import MEDIUM
    from tests.libcases import make_plan
    from tests.oracle_util import POISON, make_oracle, seeded_train_buf

    case = MEDIUM[1]
    orc = make_oracle(case)
    ranks = list(range(orc.n_ranks))
    poison = np.full(orc.gen_region_offsets(ranks)[-1], POISON, np.uint16)
    with make_plan(case, B.HF_COPY_OWN) as pl:
        ar = Arena(pl)

        def check(run, seed, what):
            print(f"[launch parameters: {what}]", flush=True)
            train = seeded_train_buf(orc, seed)
            ar.train.copy_(torch.from_numpy(train.view(np.int16)))
            ar.gen.fill_(POISON - 0x10000)
            run()
            torch.cuda.synchronize()
            assert np.array_equal(ar.gen.cpu().numpy().view(np.uint16), orc.reshard(train, poison.copy(), ranks)), what

        side = torch.cuda.Stream()  # default priority
        with torch.cuda.stream(side):
            ar.execute()  # warm-up outside capture
        side.synchronize()
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g, stream=side):
            ar.execute()
        check(g.replay, 40, "replay")
        assert pl.get_param(B.HF_PARAM_AUTOMATIC_LIST) > 0
        for i, (param, named, automatic) in enumerate([(B.HF_PARAM_CACHE_POLICY, 0, -1), (B.HF_PARAM_VARIANT, B.HF_VARIANT_PERSISTENT, B.HF_VARIANT_PARTS),
                                                       (B.HF_PARAM_WG_THREADS, 256, 0), (B.HF_PARAM_PART_BYTES, 4096, 0)]):
            pl.set_param(param, named)
            assert pl.get_param(B.HF_PARAM_AUTOMATIC_LIST) == 0
            check(ar.execute, 50 + 4 * i, f"{param} = {named}")
            check(g.replay, 51 + 4 * i, f"{param} = {named}, replay")
            pl.set_param(param, automatic)
            assert pl.get_param(B.HF_PARAM_AUTOMATIC_LIST) > 0
            check(ar.execute, 52 + 4 * i, f"{param} given back")
            check(g.replay, 53 + 4 * i, f"{param} given back, replay")
