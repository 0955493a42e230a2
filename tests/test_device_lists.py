"""The records and slots that the kernels walk (csrc/slots.hpp), against the tile lists they are
made from: every destination byte, every load inside the sources, every load-only record in front
of just the copies it is for.  Host code, under AddressSanitizer and UndefinedBehaviorSanitizer."""
import os
import shutil
import subprocess

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.mark.skipif(shutil.which("g++") is None, reason="g++ not available")
def test_device_lists_move_the_bytes_of_the_tiles(tmp_path):
    exe = str(tmp_path / "device_lists")
    csrc = os.path.join(ROOT, "paper_2409_19256_amd", "csrc")
    subprocess.run(["g++", "-std=c++17", "-O2", "-g", "-fsanitize=address,undefined", "-fno-sanitize-recover=all", "-static-libasan",
                    "-I", os.path.join(ROOT, "include"), "-I", csrc, os.path.join(csrc, "planner.cpp"),
                    os.path.join(ROOT, "tests", "device_list_main.cpp"), "-o", exe], check=True, capture_output=True, text=True)
    env = dict(os.environ, ASAN_OPTIONS="detect_leaks=1:abort_on_error=0:verify_asan_link_order=0")
    r = subprocess.run([exe], capture_output=True, text=True, env=env, timeout=300)
    assert r.returncode == 0 and r.stdout == "ok\n", r.stdout + r.stderr


@pytest.mark.gpu
@pytest.mark.parametrize("cols", [1, 2, 3, 4, 5, 6, 7, 8, 9, 15, 17, 63, 64, 65, 127, 344, 1376])
def test_rows_at_the_edges_of_slots_and_lines(cols):
    """Row-parallel stripes of 2 to 2752 bytes (every length below a slot; just below, at and above a slot of 16 bytes, a line of
    128, a wavefront's 1 KiB) and q/k/v blocks of an odd width, in every multicast mode, both
    directions and the offload image, against the oracle, whole buffers with their padding.  With the library's workgroup size,
    256 lanes for one-to-one lists as short as the way back here, and with single wavefronts, which longer ones run."""
    import torch

    from oracle.reshard_oracle import GenLayout, Model, ReshardOracle, TrainLayout
    from paper_2409_19256_amd import binding as B
    from paper_2409_19256_amd.arena import Arena
    from tests.libcases import make_plan
    from tests.oracle_util import POISON, seeded_train_buf

    poison = POISON - 0x10000
    case = dict(name="edges", model=Model(2, 71, 4, 4, 9, 4 * cols, 52), train=TrainLayout(1, 4, 1), gen=GenLayout(1, 1))
    orc = ReshardOracle(case["model"], case["train"], case["gen"])
    ranks = list(range(orc.n_ranks))
    train = seeded_train_buf(orc, 900 + cols)
    empty = np.full(orc.gen_region_offsets(ranks)[-1], POISON, np.uint16)
    want = orc.reshard(train, empty.copy(), ranks)
    back = orc.reshard_back(want, ranks, np.full(train.shape, POISON, np.uint16))
    for mode, threads in [(m, n) for m in (B.HF_MULTICAST_OFF, B.HF_MULTICAST_REGISTERS, B.HF_MULTICAST_CACHE_BLOCKED, B.HF_MULTICAST_PREFETCHED)
                          for n in (0, 64)]:
        print(f"[edges cols {cols} mode {mode} lanes {threads}]", flush=True)
        with make_plan(case, B.HF_COPY_OWN) as pl:
            pl.set_param(B.HF_PARAM_MULTICAST, mode)
            pl.set_param(B.HF_PARAM_WG_THREADS, threads)
            if threads == 0:
                assert pl.bytes_moved(1) + pl.unique_src_bytes(1) <= 24 << 20  # the way back: 256 lanes
            ar = Arena(pl)
            ar.train.copy_(torch.from_numpy(train.view(np.int16)))
            ar.gen.fill_(poison)
            ar.execute()
            torch.cuda.synchronize()
            assert np.array_equal(ar.gen.cpu().numpy().view(np.uint16), want)
            ar.train.fill_(poison)
            ar.back()
            torch.cuda.synchronize()
            assert np.array_equal(ar.train.cpu().numpy().view(np.uint16), back)
    with make_plan(case, B.HF_PLAN_OFFLOAD) as pl:
        total = pl.remote_bytes // 2
        image = torch.full((total,), poison, dtype=torch.int16, pin_memory=True)
        gen = torch.from_numpy(want.view(np.int16)).cuda()
        st = Arena.stream_handle()
        pl.offload_remote(gen.data_ptr(), image.data_ptr(), st)
        torch.cuda.synchronize()
        assert np.array_equal(image.numpy().view(np.uint16), orc.pack_remote(want, ranks, np.full(total, POISON, np.uint16)))
        tags = orc.owner_tags(ranks)
        lost = want.copy()
        for i, r in enumerate(ranks):
            lo, hi = orc.gen_region_offsets(ranks)[i:i + 2]
            lost[lo:hi][(tags[lo:hi] >= 0) & (tags[lo:hi] != r)] = 0x0BAD
        gen.copy_(torch.from_numpy(lost.view(np.int16)))
        pl.reload_remote(image.data_ptr(), gen.data_ptr(), st)
        torch.cuda.synchronize()
        assert np.array_equal(gen.cpu().numpy().view(np.uint16), want)
