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
    w1 = sy.shrink(sy.WORKLOADS["tiny_f32"], batch=1, n_q_heads=64, n_kv_heads=1, head_dim=128, seq=128, n_bswa_chunks=1)
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


@pytest.mark.parametrize("io,d,C,rows,heads,many", [
    ("f32", 64, 40, 40, (2, 2), 20), ("f32", 64, 72, 100, (2, 2), 60),        # workgroups beyond the line for states of up to 64 rows, of more
    ("bf16", 64, 40, 33, (2, 1), 16), ("bf16", 64, 72, 100, (2, 2), 16),
    ("bf16", 128, 40, 64, (1, 1), 6), ("bf16", 128, 72, 100, (4, 2), 24),
    ("f32", 128, 256, 256, (4, 4), 16),                                       # attention long enough to hide the folds
])
def test_a_sequence_among_many(io, d, C, rows, heads, many):
    """Alone a sequence has a chunk's scores taken along by its attention launch, among many in a launch of their own or
    beside attention: the same outputs, state and record to the bit."""
    import torch
    import paper_2605_09877_amd as pkg
    from paper_2605_09877_amd import synth as sy
    w = sy.shrink(sy.WORKLOADS["tiny_f32"], io=io, batch=many, n_q_heads=heads[0], n_kv_heads=heads[1], head_dim=d, seq=C * 6 + 5, chunk_len=C,
                  budget_kind="table", budget_table=(rows, rows, rows, rows + 20, rows + 20, rows + 21))
    q, k, v = sy.make_qkv(w, "cuda:0")
    res = []
    for n in (1, many):
        st = pkg.state_for(sy.shrink(w, batch=n), device="cuda:0")
        assign, score = st.trace(6)
        out, lse = st.prefill(*(x[:n].contiguous() for x in (q, k, v)), want_lse=True)
        state = st.export()
        nf = st.folds
        res.append([x[0] for x in (out, lse)] + [x[:nf, 0] for x in (assign, score.view(torch.int32))] +
                   [state[key][0] for key in ("sK", "sV", "n", "khat", "vhat")])
    for i, (one, among) in enumerate(zip(*res)):
        assert torch.equal(one, among), i
