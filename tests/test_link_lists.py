"""Offload and reload where a workgroup's batches run on from one record into the next: one workgroup for all records, as many as
records, more; records of one batch and of several; rows of 14 bytes, which take the other kernel.  Against the oracle's image."""
import numpy as np
import pytest


@pytest.mark.gpu
@pytest.mark.parametrize("cols", [7, 8, 33, 640])
@pytest.mark.parametrize("tile_bytes,wgs", [(4096, 1), (4096, 2), (4096, 3), (4096, 4096), (32768, 1), (131072, 1), (131072, 7), (131072, 64)])
def test_batches_run_on_across_records(cols, tile_bytes, wgs):
    import torch

    from oracle.reshard_oracle import GenLayout, Model, ReshardOracle, TrainLayout
    from paper_2409_19256_amd import binding as B
    from tests.libcases import make_plan
    from tests.oracle_util import POISON, seeded_train_buf

    print(f"[link cols {cols} tile {tile_bytes} wgs {wgs}]", flush=True)
    case = dict(name="link", model=Model(2, 136, 4, 4, 9, 4 * cols, 1204), train=TrainLayout(1, 4, 1), gen=GenLayout(1, 1))
    orc = ReshardOracle(case["model"], case["train"], case["gen"])
    ranks = [2, 0]
    train = seeded_train_buf(orc, 300 + cols)
    gen = orc.reshard(train, np.full(orc.gen_region_offsets(ranks)[-1], POISON, np.uint16), ranks)
    tags = orc.owner_tags(ranks)
    lost = gen.copy()
    for i, r in enumerate(ranks):
        lo, hi = orc.gen_region_offsets(ranks)[i:i + 2]
        lost[lo:hi][(tags[lo:hi] >= 0) & (tags[lo:hi] != r)] = 0x0BAD
    with make_plan(case, B.HF_PLAN_OFFLOAD, mat=ranks) as pl:
        pl.set_param(B.HF_PARAM_TILE_BYTES, tile_bytes)
        pl.set_param(B.HF_PARAM_OFFLOAD_WGS, wgs)
        total = pl.remote_bytes // 2
        image = torch.full((total,), POISON - 0x10000, dtype=torch.int16, pin_memory=True)
        buf = torch.from_numpy(gen.view(np.int16)).cuda()
        st = torch.cuda.current_stream().cuda_stream
        pl.offload_remote(buf.data_ptr(), image.data_ptr(), st)
        torch.cuda.synchronize()
        assert np.array_equal(image.numpy().view(np.uint16), orc.pack_remote(gen, ranks, np.full(total, POISON, np.uint16)))
        buf.copy_(torch.from_numpy(lost.view(np.int16)))
        pl.reload_remote(image.data_ptr(), buf.data_ptr(), st)
        torch.cuda.synchronize()
        assert np.array_equal(buf.cpu().numpy().view(np.uint16), gen)
