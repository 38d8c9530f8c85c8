"""The append selection of folds that are a kernel per step, against the rule applied to the scores that the library
recorded: the tokens with the smallest (score, position) become rows, in position order.  Blocks that are not a
multiple of 64 tokens, of one piece of 64 and of many, appends of 17 tokens (the fewest that have a launch of their
own), a piece's edge and all but one, and scores that are equal (copies of a token, of which the earliest are taken)."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("io", ["f32", "bf16"])
@pytest.mark.parametrize("C,appends", [(40, (17, 39)), (64, (63, 17)), (65, (64, 0, 17)), (130, (17, 129)), (520, (33, 1, 519)),
                                       (1100, (1099, 64))])
def test_selection_follows_the_recorded_scores(C, appends, io):
    import paper_2605_09877_amd as pkg
    from paper_2605_09877_amd import binding as b
    from paper_2605_09877_amd import synth as sy
    rows = [C, C]    # after the first chunk, after the second (which creates the state)
    for n in appends:
        rows.append(rows[-1] + n)
    w = sy.shrink(sy.WORKLOADS["tiny_f32"], io=io, batch=2, n_q_heads=2, n_kv_heads=2, chunk_len=C, seq=C * len(rows), rope_dims=16,
                  budget_kind="table", budget_table=tuple(rows))
    q, k, v = sy.make_qkv(w, "cuda:0")
    for c in range(len(rows)):   # every block: its first half again
        k[:, c * C + C // 2:c * C + C // 2 * 2] = k[:, c * C:c * C + C // 2]
    params = sy.make_params(w, "cuda:0", plain=False)
    st = pkg.state_for(w, device="cuda:0", **params)
    st.debug_set(b.KVM_DEBUG_FOLD_PATH, 2)
    assign, score = st.trace(len(rows))
    st.prefill(q, k, v, params["gate"])
    torch.cuda.synchronize()
    assign, score = assign.cpu().numpy(), score.cpu().numpy()
    assert st.folds == len(rows) - 1 and st.rows == rows[-1]
    for f, n in enumerate(appends, start=1):
        for unit in np.ndindex(2, 2):
            s, to = score[f][unit], assign[f][unit]
            appended = np.nonzero(np.isnan(s[:, 1]))[0]
            want = np.sort(np.lexsort((np.arange(C), s[:, 0]))[:n])
            assert np.array_equal(appended, want), (f, unit)
            assert np.array_equal(to[appended], rows[f] + np.arange(n)), (f, unit)
