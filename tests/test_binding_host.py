"""The binding's host side, without a GPU: who owns the memory that calls hand to the library."""
import torch

from paper_2605_09877_amd import binding as kb


def test_a_table_that_is_written_belongs_to_one_call():
    """More than 64 states: kvm_decode_step_multi writes its workspace and its kernels read it, so no two calls that may be
    under way together have the same one, and none outlives its call.  Up to 64 it is never touched, and kept."""
    dev = torch.device("cpu")
    held = [kb._multi_workspace(dev, 65 * 56, 65) for _ in range(3)]
    assert len({ws.data_ptr() for ws in held}) == 3 and all(ws.numel() == 65 * 56 for ws in held)
    kept = kb._multi_workspace(dev, 64 * 56, 64)
    assert all(kept.data_ptr() != ws.data_ptr() for ws in held)
    assert kb._multi_workspace(dev, 7 * 56, 7) is kept
    assert kb._multi_workspace(dev, 4096 * 56, 64).numel() >= 4096 * 56   # 64 states of many sequences
