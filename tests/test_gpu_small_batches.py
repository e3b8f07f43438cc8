"""A candidate evaluated alone, where several workgroups share it and the products are spread over 32 x 32 tiles, and as
the first of a batch that fills the chip, where neither is so: the same bits."""
import numpy as np
import pytest

from paper_2209_12769_amd import workloads as wl

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def B():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2209_12769_amd import binding
    binding.lib()
    return binding


def _predictions(B, model, g, labs):
    w = wl.with_time_like_head(wl.custom("small", model, [g], [labs], seed=11))
    ev = B.evaluator_for(w)
    cg, co, gid = ev.to_device(w.cand_graph), ev.to_device(w.cand_off), ev.to_device(w.group_id)
    pred = ev.eval_candidates(cg, co, gid).cpu().numpy()
    assert ev.check() == B.DC_OK
    ev.close()
    return pred


# fp32: H = 32, 96 and 160 (tiles of 32 columns), 64 and 192 (general kernel), 128, 256, 384 (pipelined kernel)
@pytest.mark.parametrize("F,H,L,dtype", [(16, 32, 2, "f32"), (48, 96, 2, "f32"), (16, 160, 1, "f32"), (32, 64, 2, "f32"),
                                         (16, 192, 1, "f32"), (32, 128, 3, "f32"), (64, 256, 2, "f32"), (80, 384, 1, "f32"),
                                         (64, 256, 4, "bf16")])
def test_alone_and_first_of_a_full_batch(B, F, H, L, dtype):
    model = wl.ModelSpec(F, H, L, dtype)
    for n, p, C in ((1, 0.0, 2100), (33, 0.1, 2100), (257, 0.02, 700)):
        g = wl.random_dag(900 + n, n, p, F)
        one = np.concatenate([wl.random_labels(n, g.n, max(1, n - 2), C=1), np.arange(g.n, dtype=np.int32)[None]])
        for lab in one:
            alone = _predictions(B, model, g, lab[None])
            print(F, H, L, dtype, n, C, flush=True)
            many = _predictions(B, model, g, np.tile(lab, (C, 1)))
            assert alone[0] == many[0]
            assert dtype == "bf16" or np.all(many == many[0])
