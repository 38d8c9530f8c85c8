"""Prompts of states without the matrix-core folds, chunk by chunk: the scores of a chunk's fold come from workgroups of its
attention launch, memory keys of up to eight blocks from one launch.  Against the CPU oracle: one block more and one
less than a launch of keys, blocks that four tokens do not divide, states of less and more than 128 rows (two rows of a
lane), blocks from the ring, head_dim 64 on either side of the matrix cores, appends that need no scores and some."""
import pytest

from test_gpu_parity import run_prefill_case

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("io,d,C,rows,blocks,tail,heads,split", [
    ("f32", 64, 64, 64, 9, 0, (2, 2), None),
    ("f32", 64, 30, 129, 10, 7, (4, 2), 60),
    ("f32", 128, 33, 65, 11, 1, (1, 1), 33 * 3),
    ("f32", 128, 64, 193, 8, 33, (2, 1), None),
    ("bf16", 64, 64, 127, 10, 5, (4, 1), 128),
    ("bf16", 64, 50, 130, 9, 3, (2, 2), None),      # a block the tiles do not divide
    ("bf16", 128, 40, 257, 12, 9, (2, 1), 80),
])
@pytest.mark.parametrize("batch", [1, 5])
def test_prefill_against_the_oracle(io, d, C, rows, blocks, tail, heads, split, batch):
    from paper_2605_09877_amd import synth as sy
    w = sy.shrink(sy.WORKLOADS["tiny_f32"], io=io, batch=batch, n_q_heads=heads[0], n_kv_heads=heads[1], head_dim=d, rope_dims=16,
                  seq=C * blocks + tail, chunk_len=C, budget_fixed=rows)
    run_prefill_case(w, plain=False, split=split, units=[(0, 0), (batch - 1, heads[1] - 1)],
                     case=f"chunk_by_chunk[{io},{d},{C},{rows},{batch}]")


@pytest.mark.parametrize("batch", [4064, 4096])
def test_more_workgroups_than_a_dimension_holds(batch):
    """64 heads x 64 queries x 4096 sequences are 2^24 attention workgroups: with those of the scores beside them (4064: just
    below, 4096: above) more than one dimension of a launch takes.  Every sequence has the inputs, and so the bits, of
    one alone."""
    import torch
    import paper_2605_09877_amd as pkg
    from paper_2605_09877_amd import synth as sy
    w1 = sy.shrink(sy.WORKLOADS["tiny_f32"], batch=1, n_q_heads=64, n_kv_heads=1, seq=128, n_bswa_chunks=1)
    qkv = sy.make_qkv(w1, "cuda:0")
    res = []
    for n in (1, batch):
        st = pkg.state_for(sy.shrink(w1, batch=n), device="cuda:0")
        out = st.prefill(*(x.expand(n, -1, -1, -1) for x in qkv))
        state = st.export()
        assert st.folds == 2 and st.rows == 64
        res.append((out, *(state[key] for key in ("sK", "sV", "n", "khat", "vhat"))))
    for one, many in zip(*res):
        assert bool((many == one).all())
