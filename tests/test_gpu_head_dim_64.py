"""Prompts in bf16 with head_dim 64 (attention on the matrix cores, folds by the generic kernels) against the CPU
oracle: block lengths of one tile and several, state sizes inside and at the ends of a tile, query heads
that share a workgroup and that do not, keys from the window ring, ragged ends, temperatures of every
sign.  Bars are the oracle's for bf16 (kvm_testlib.check_outputs)."""
import pytest

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
