"""Lists short enough for larger workgroups, and lists just too long for them: the library's own choice leaves the same bytes as
single wavefronts over the named list, which the parity tests compare with the oracle."""
import pytest
import torch

from paper_2409_19256_amd import Plan, binding as B

pytestmark = pytest.mark.gpu

# hidden, heads, head dim, ffn, vocab; train (p, t, d), generation (p_g, t_g); layers below and above the line
SHAPES = {
    "whole_lines": ((512, 8, 64, 1408, 512), (1, 2, 1), (1, 1), (1, 2)),        # 24 MiB of one-to-one copies lie between
    "rows_of_260_bytes": ((260, 4, 65, 896, 548), (1, 2, 1), (1, 1), (6, 7)),
    "rows_of_14_bytes": ((56, 4, 14, 28, 64), (1, 4, 1), (1, 2), (1, 3)),       # always short, rows below a slot
    "three_destinations": ((256, 4, 64, 704, 512), (1, 4, 1), (1, 1), (4, 6)),  # 32 MiB of shared pieces (seven: 64) lie between
    "three_destinations_joined": ((384, 4, 96, 1324, 512), (1, 4, 1), (1, 1), (1, 2)),
    "seven_destinations": ((256, 8, 32, 712, 512), (1, 8, 1), (1, 1), (3, 6)),
}


def _random(n, seed):
    gen = torch.Generator(device="cuda").manual_seed(seed)
    return torch.randint(-32768, 32768, (n,), generator=gen, dtype=torch.int16, device="cuda")


@pytest.mark.parametrize("layers", [0, 1], ids=["below", "above"])
@pytest.mark.parametrize("name", SHAPES)
def test_larger_workgroups_move_the_same_bytes(name, layers):
    (h, heads, hd, ffn, vocab), train, gen, depth = SHAPES[name]
    print(f"[{name} {depth[layers]} layers]", flush=True)
    model = dict(n_layers=depth[layers], hidden=h, n_q_heads=heads, n_kv_heads=heads, head_dim=hd, ffn=ffn, vocab=vocab)
    for flags in (B.HF_SKIP_OWN, B.HF_COPY_OWN, B.HF_GATHER_FROM_GEN):
        with Plan(model, train, gen, flags=flags) as plan:
            a, b = _random(plan.train_bytes // 2, 1), _random(plan.gen_bytes // 2, 2)
            results = []
            for threads in (0, 64):                              # 64: the list of the mode in force, one wavefront per KiB
                plan.set_param(B.HF_PARAM_WG_THREADS, threads)
                t, g = a.clone(), b.clone()
                plan.execute(t.data_ptr(), g.data_ptr())
                if not flags & B.HF_GATHER_FROM_GEN:
                    plan.install_own(t.data_ptr(), g.data_ptr())
                out = torch.full_like(a, 0x5A5A)
                plan.back(out.data_ptr(), g.data_ptr())
                torch.cuda.synchronize()
                results.append((t, g, out))
            assert torch.equal(results[0][0], a)
            for x, y in zip(*results):
                assert torch.equal(x, y)
