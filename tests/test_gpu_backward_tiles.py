"""The backward pass on the matrix cores at the edges of its tiles: 32-query and 64-key tiles, 128-key workgroups,
one and several heads per KV head; a chunk's roles in one launch and in several, D formed inside dq and by a pass ahead of the
walk.  Oracle and bars of test_gpu_backward."""
import pytest
import torch

from test_gpu_backward import run_backward_case

pytestmark = pytest.mark.gpu


def workgroups(units, heads, C, rows):
    """Of a whole chunk (dq, window keys, state rows), and of those that count for where D is formed (dq, state rows)."""
    eights, G, win, st = (units + 7) // 8 * 8, heads[0] // heads[1], (C + 127) // 128, (rows + 127) // 128
    return eights * (G * win + win + st), units * (G * win + st)


def one_launch(units, heads, C, rows):
    return workgroups(units, heads, C, rows)[0] <= (1024 if heads[0] <= 2 * heads[1] else 256)


@pytest.mark.parametrize("C,rows,T,heads", [
    (64, 65, 64 * 4 + 1, (1, 1)),        # one query in the last tile, one state row beyond a tile
    (64, 127, 64 * 5 + 33, (3, 1)),      # a query beyond a 32-row tile, three heads streamed one after the other
    (128, 129, 128 * 4 + 31, (4, 2)),    # a workgroup with one state row
    (192, 200, 192 * 3 + 95, (2, 2)),    # the block's second workgroup half empty
    (256, 256, 256 * 3 + 1, (2, 1)),
    (256, 300, 256 * 4, (4, 1)),
])
@pytest.mark.parametrize("launches", [1, 2, 3])   # one; several, D inside dq; several, D ahead
def test_tile_edges(C, rows, T, heads, launches):
    from paper_2605_09877_amd import binding as b
    from paper_2605_09877_amd import synth as sy
    w = sy.shrink(sy.WORKLOADS["prefill_fixed"], batch=1, n_q_heads=heads[0], n_kv_heads=heads[1], seq=T, chunk_len=C,
                  budget_fixed=rows)
    run_backward_case(w, plain=False, knobs={b.KVM_DEBUG_BACKWARD_LAUNCHES: launches})


@pytest.mark.parametrize("heads,many,ahead", [((2, 2), 90, False), ((4, 1), 30, True)])
def test_gradients_do_not_depend_on_the_batch(heads, many, ahead):
    """Alone a sequence's chunks are one launch each, among many several: with D formed inside dq, or ahead of the walk.
    The same gradients to the bit."""
    import paper_2605_09877_amd as kvm
    assert one_launch(heads[1], heads, 256, 256) and not one_launch(many * heads[1], heads, 256, 256)
    assert (workgroups(many * heads[1], heads, 256, 256)[1] <= 512) == ahead
    gen = torch.Generator(device="cuda:0").manual_seed(3)
    mk = lambda h: torch.randn(many, 256 * 3 + 1, h, 128, generator=gen, device="cuda:0").bfloat16()
    q, k, v, dout = mk(heads[0]), mk(heads[1]), mk(heads[1]), mk(heads[0])

    def grads(n):
        leaves = [x[:n].contiguous().requires_grad_(True) for x in (q, k, v)]
        out = kvm.kvm_attention(*leaves, chunk_len=256, rope_dims=32, budget_fixed=256)
        return (out.detach(),) + torch.autograd.grad(out, leaves, dout[:n].contiguous())

    for one, all_ in zip(grads(1), grads(many)):
        assert torch.equal(one[0], all_[0])


@pytest.mark.parametrize("heads,many", [((2, 2), 200), ((2, 1), 272), ((4, 1), 70), ((4, 1), 48)])
@pytest.mark.parametrize("C,rows", [(64, 70), (256, 256)])
def test_gradients_of_one_launch_and_of_several(heads, many, C, rows):
    """A sequence alone, whose chunks are one launch each, and the same one among so many that they are not: the same
    gradients to the bit."""
    import paper_2605_09877_amd as kvm
    assert one_launch(heads[1], heads, C, rows) and not one_launch(many * heads[1], heads, C, rows)
    gen = torch.Generator(device="cuda:0").manual_seed(5)
    mk = lambda h: torch.randn(many, C * 3 + 33, h, 128, generator=gen, device="cuda:0").bfloat16()
    q, k, v, dout = mk(heads[0]), mk(heads[1]), mk(heads[1]), mk(heads[0])

    def grads(n):
        leaves = [x[:n].contiguous().requires_grad_(True) for x in (q, k, v)]
        out = kvm.kvm_attention(*leaves, chunk_len=C, rope_dims=32, budget_fixed=rows)
        return (out.detach(),) + torch.autograd.grad(out, leaves, dout[:n].contiguous())

    for one, all_ in zip(grads(1), grads(many)):
        assert torch.equal(one[0], all_[0])
