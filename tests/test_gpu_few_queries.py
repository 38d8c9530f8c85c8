"""Prefill attention on the matrix cores on both sides of the line between the kernel whose waves share 32 queries and split
their keys (up to 64 workgroups of the other one, 128 with head_dim 64) and the one whose waves share the keys, against the CPU oracle: state
sizes around a 32-row tile, last chunks of 1, 31, 32 and 33 queries, fewer tiles than waves, keys from the ring,
heads that share keys, temperatures of every sign.  Bars are the oracle's for bf16 (kvm_testlib.check_outputs)."""
import pytest

from test_gpu_parity import run_prefill_case

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("many", [False, True])
@pytest.mark.parametrize("d", [128, 64])
@pytest.mark.parametrize("C,rows,tail,heads,split,signs", [
    (64, 64, 1, (1, 1), None, (1, 1)),         # two tiles of window, one query in the last chunk
    (64, 65, 31, (4, 1), None, (-1, 1)),       # a row beyond a tile; heads that share keys
    (64, 95, 33, (2, 1), 128, (1, -1)),        # a row short of a tile; the second call's window is in the ring
    (128, 129, 32, (3, 3), 256, (-1, -1)),
    (192, 223, 64, (8, 2), None, (1, 1)),      # blocks of six 32-query pieces
])
def test_prefill_against_the_oracle(C, rows, tail, heads, split, signs, d, many):
    from paper_2605_09877_amd import synth as sy
    batch = 1 + 1024 // (C * heads[0])         # (head_dim 64: the fewest queries that go to the matrix cores)
    if many:
        batch += 8 * 128 // heads[0]
    w = sy.shrink(sy.WORKLOADS["prefill_fixed"], batch=batch, n_q_heads=heads[0], n_kv_heads=heads[1], head_dim=d, rope_dims=16,
                  seq=4 * C + tail, chunk_len=C, budget_fixed=rows)

    def tweak(params):
        params["tau_state"] *= signs[0]
        params["tau_bswa"] *= signs[1]

    run_prefill_case(w, plain=False, split=split, tweak=tweak, units=[(0, 0), (batch - 1, heads[1] - 1)],
                     case=f"few_queries[{C},{rows},{tail},{heads},{d},{many}]")


@pytest.mark.parametrize("C,rows,T,heads", [(64, 70, 64 * 6 + 9, (4, 1)), (256, 300, 256 * 4 + 70, (2, 2)), (192, 192, 192 * 5, (1, 1))])
@pytest.mark.parametrize("scale", [1.0, 12.0])   # 12: maxima that rise by far more than the exponentials' slack
def test_outputs_do_not_depend_on_the_batch(C, rows, T, heads, scale):
    """head_dim 128: a sequence alone and the same one among many, the other kernel's, have equal bits."""
    import torch
    import paper_2605_09877_amd as pkg
    from paper_2605_09877_amd import synth as sy
    many = 1 + 8 * 128 // heads[0]
    w = sy.shrink(sy.WORKLOADS["prefill_fixed"], batch=many, n_q_heads=heads[0], n_kv_heads=heads[1], seq=T, chunk_len=C, budget_fixed=rows)
    q, k, v = sy.make_qkv(w, "cuda:0")
    q *= scale
    res = []
    for n in (many, 1):
        wn = sy.shrink(w, batch=n)
        st = pkg.state_for(wn, device="cuda:0", **sy.make_params(wn, "cuda:0", plain=True))
        res.append([x[0].clone() for x in st.prefill(q[:n].contiguous(), k[:n].contiguous(), v[:n].contiguous(), want_lse=True)])
    assert torch.equal(res[0][0], res[1][0]) and torch.equal(res[0][1], res[1][1])


@pytest.mark.parametrize("where", ["v", "k"])
@pytest.mark.parametrize("value", [float("nan"), float("inf")])
@pytest.mark.parametrize("C,heads,back", [(64, (4, 1), 5), (128, (2, 2), 70), (256, (4, 2), 1)])
@pytest.mark.parametrize("many", [False, True])
def test_a_value_that_is_not_finite_stays_within_64_positions(C, heads, back, value, where, many):
    """head_dim 128, either kernel: a token of the last block, `back` tokens from the prompt's end, holds a value that is not
    finite.  Queries of earlier 64 positions, other channels of v, other heads and sequences have the bits that they have
    without it.  With k the 32 queries of its piece share the reference point of their exponentials p, which then moves: p are
    rounded to bf16 from another scale, 2^-9 of each at most, either time, so that their sum, in lse, is off by 2^-8
    and the output, a mean of v weighted by them, by 2^-8 of the largest v, beside its own two roundings."""
    import torch
    import paper_2605_09877_amd as pkg
    from paper_2605_09877_amd import synth as sy
    T, batch, G = C * 4 - 3, 1 + many * (8 * 128 // heads[0]), heads[0] // heads[1]
    tiles = (batch * heads[1] + 7) // 8 * 8 * (C // 32 * (G // 4) if G % 4 == 0 else (C + 127) // 128 * G)
    assert (tiles > 64) == many
    w = sy.shrink(sy.WORKLOADS["prefill_fixed"], batch=batch, n_q_heads=heads[0], n_kv_heads=heads[1], rope_dims=16, seq=T, chunk_len=C,
                  budget_fixed=2 * C)
    q, k, v = sy.make_qkv(w, "cuda:0")
    params = sy.make_params(w, "cuda:0", plain=False)

    def run(k, v):
        st = pkg.state_for(w, device="cuda:0", **params)
        return st.prefill(q, k, v, params["gate"], want_lse=True)

    at = T - back
    want, want_lse = run(k, v)
    k2, v2 = k.clone(), v.clone()
    (k2 if where == "k" else v2)[0, at, 0, 3] = value
    out, lse = run(k2, v2)
    assert torch.equal(out[:, :, G:], want[:, :, G:]) and torch.equal(out[1:], want[1:])
    assert torch.equal(lse[:, :at // 32 * 32], want_lse[:, :at // 32 * 32]) and torch.equal(out[:, :at // 64 * 64], want[:, :at // 64 * 64])
    if where == "v":
        others = [c for c in range(128) if c != 3]
        assert torch.equal(lse, want_lse) and torch.equal(out[..., others], want[..., others])
        assert not out[0, at:, :G, 3].isfinite().any()
    else:
        torch.testing.assert_close(out[:, :at].float(), want[:, :at].float(), rtol=2 ** -8, atol=2 ** -8 * float(v.abs().max()))
        torch.testing.assert_close(lse[:, :at], want_lse[:, :at], rtol=1e-5, atol=2 ** -8)
