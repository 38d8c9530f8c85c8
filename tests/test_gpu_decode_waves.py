"""Decode steps on both sides of the line between workgroups of eight waves (as many (sequence, head group) pairs as compute
units, 256, or fewer, but more than share their keys) and of four, with fewer keys than a round of the waves and more,
folds among them, against the CPU oracle; the same tokens in states of their own, one launch for all."""
import pytest
import torch

from test_gpu_parity import run_prefill_case

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("io,d,batch,heads", [
    ("bf16", 128, 64, (16, 4)), ("bf16", 128, 65, (16, 4)),     # 256 and 260 pairs of four heads
    ("bf16", 128, 43, (6, 3)), ("bf16", 64, 129, (4, 2)),       # 129 and 258 pairs of two
    ("bf16", 64, 130, (1, 1)), ("f32", 64, 256, (1, 1)), ("f32", 128, 129, (2, 2)),
])
@pytest.mark.parametrize("rows", [64, 200])
def test_decode_against_the_oracle(io, d, batch, heads, rows):
    from paper_2605_09877_amd import synth as sy
    w = sy.shrink(sy.WORKLOADS["tiny_f32"], io=io, batch=batch, n_q_heads=heads[0], n_kv_heads=heads[1], head_dim=d, rope_dims=16,
                  seq=64 * 5 + 9, chunk_len=64, budget_fixed=rows)
    run_prefill_case(w, plain=False, decode_tail=64 + 11, units=[(0, 0), (batch - 1, heads[1] - 1)],
                     case=f"decode_waves[{io},{d},{batch},{rows}]")


@pytest.mark.parametrize("n", [64, 65])
def test_states_of_their_own_agree_with_one_state(n):
    """n sequences as n states of one, decode_multi, and as one state of n, decode: the same workgroups, the same bits."""
    import paper_2605_09877_amd as pkg
    from paper_2605_09877_amd import synth as sy
    from paper_2605_09877_amd.binding import decode_multi
    w = sy.shrink(sy.WORKLOADS["prefill_fixed"], batch=n, n_q_heads=8, n_kv_heads=4, chunk_len=64, seq=64 * 3, budget_fixed=128)
    q, k, v = sy.make_qkv(w, "cuda:0")
    cut = lambda x, i: x[i:i + 1, :128].contiguous()
    one = pkg.state_for(w, device="cuda:0", **sy.make_params(w, "cuda:0", plain=True))
    one.prefill(q[:, :128].contiguous(), k[:, :128].contiguous(), v[:, :128].contiguous())
    w1 = sy.shrink(w, batch=1)
    many = [pkg.state_for(w1, device="cuda:0", **sy.make_params(w1, "cuda:0", plain=True)) for _ in range(n)]
    for i, st in enumerate(many):
        st.prefill(cut(q, i), cut(k, i), cut(v, i))
    for t in range(128, w.seq):
        tok = [x[:, t].contiguous() for x in (q, k, v)]
        assert torch.equal(one.decode(*tok), decode_multi(many, *tok)), t
