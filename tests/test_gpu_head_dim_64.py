"""Prompts in bf16 with head_dim 64 (attention on the matrix cores, folds by the generic kernels) against the CPU
oracle: block lengths of one tile and several, state sizes inside and at the ends of a tile, query heads
that share a workgroup and that do not, keys from the window ring, ragged ends, temperatures of every
sign.  Bars are the oracle's for bf16 (kvm_testlib.check_outputs)."""
import pytest
import torch

from test_gpu_parity import run_prefill_case

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("C,rows,T,heads,split", [
    (64, 64, 64 * 3 + 1, (1, 1), None),        # one tile a block, one query in the last
    (64, 65, 64 * 6 + 63, (4, 1), None),       # a row beyond the tile; four heads share a workgroup
    (64, 127, 64 * 5, (6, 3), 128),          # two heads a group; the second call's window is in the ring
    (128, 129, 128 * 4 + 33, (8, 1), 256),
    (192, 200, 192 * 3 + 95, (2, 2), None),    # tiles per block not a power of two
    (256, 320, 256 * 4 + 129, (12, 3), 768),
    (96, 160, 96 * 5 + 7, (2, 1), None),       # a block the tiles do not divide: the row kernel
])
@pytest.mark.parametrize("signs", [(1, 1), (-1, 1), (1, -1)])
def test_prefill_against_the_oracle(C, rows, T, heads, split, signs):
    from paper_2605_09877_amd import synth as sy
    batch = 1024 // (C * heads[0]) + 1   # the fewest queries a launch takes to the matrix cores
    w = sy.shrink(sy.WORKLOADS["prefill_fixed"], batch=batch, n_q_heads=heads[0], n_kv_heads=heads[1], head_dim=64,
                  rope_dims=16, seq=T, chunk_len=C, budget_fixed=rows)

    def tweak(params):
        params["tau_state"] *= signs[0]
        params["tau_bswa"] *= signs[1]

    run_prefill_case(w, plain=False, split=split, tweak=tweak, units=[(0, 0), (batch - 1, heads[1] - 1)],
                     case=f"head_dim_64[{C},{rows},{T},{heads},{signs}]")


@pytest.mark.parametrize("where", ["v", "k"])
@pytest.mark.parametrize("value", [float("nan"), float("inf"), float("-inf")])
@pytest.mark.parametrize("C,heads,back,split", [(64, (4, 1), 5, None), (128, (8, 8), 70, None), (256, (4, 2), 1, 512)])
@pytest.mark.parametrize("many", [False, True])   # up to 128 workgroups of the tile kernel: the one whose waves split the keys; more
def test_a_value_that_is_not_finite_reaches_only_the_queries_that_see_it(C, heads, back, split, value, where, many):
    """One token of the last block, `back` tokens from the prompt's end, holds a value that is not finite (a padded tail).
    Queries before it, of the same 64-key tile too, are what they are without it, up to the two results' bf16
    rounding (2^-8 of the element each) and 1e-5 for sums in another order; queries from it on see it."""
    import paper_2605_09877_amd as pkg
    from paper_2605_09877_amd import synth as sy
    T, batch = C * 4 - 3, 1024 // (C * heads[0]) + 1 + many * (8 * 128 // heads[0])
    G = heads[0] // heads[1]
    tiles = (batch * heads[1] + 7) // 8 * 8 * (C // 32 * (G // 4) if G % 4 == 0 else (C + 127) // 128 * G)
    assert (tiles > 128) == many
    w = sy.shrink(sy.WORKLOADS["prefill_fixed"], batch=batch, n_q_heads=heads[0], n_kv_heads=heads[1], head_dim=64, rope_dims=16,
                  seq=T, chunk_len=C, budget_fixed=2 * C)
    q, k, v = sy.make_qkv(w, "cuda:0")
    params = sy.make_params(w, "cuda:0", plain=False)

    def run(k, v):
        st = pkg.state_for(w, device="cuda:0", **params)
        cuts = [0, T] if split is None else [0, split, T]
        parts = [st.prefill(*(x[:, lo:hi].contiguous() for x in (q, k, v, params["gate"])), want_lse=True)
                 for lo, hi in zip(cuts, cuts[1:])]
        return tuple(torch.cat(x, dim=1).float() for x in zip(*parts))

    at = T - back
    want, want_lse = run(k, v)
    k2, v2 = k.clone(), v.clone()
    (k2 if where == "k" else v2)[0, at, 0, 3] = value
    out, lse = run(k2, v2)
    torch.testing.assert_close(out[:, :at], want[:, :at], rtol=2 ** -7, atol=1e-5)
    torch.testing.assert_close(lse[:, :at], want_lse[:, :at], rtol=1e-5, atol=1e-5)
    assert torch.equal(out[:, :, G:], want[:, :, G:]) and torch.equal(out[1:], want[1:])   # other heads and sequences
    if where == "v":
        assert not out[0, at:, :G, 3].isfinite().any()
        torch.testing.assert_close(lse, want_lse, rtol=1e-5, atol=1e-5)
