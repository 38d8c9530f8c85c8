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


def test_a_torch_without_device_support_imports_the_host_side():
    """Sizes and schedules are the library's host code: the package imports, and answers, where torch's C layer has no
    device functions (a build for CPUs alone), and asks torch's public ones there."""
    import os
    import subprocess
    import sys
    root = os.path.dirname(os.path.dirname(os.path.abspath(kb.__file__)))
    program = (
        "import torch\n"
        "for name in ('_cuda_getDevice', '_cuda_getCurrentRawStream'):\n"
        "    if hasattr(torch._C, name):\n"
        "        delattr(torch._C, name)\n"
        "import ctypes\n"
        "import paper_2605_09877_amd as kvm\n"
        "from paper_2605_09877_amd import binding as kb\n"
        "c = kb.kvm_config(1, 2, 2, 64, 16, 64, 2, 1, kb.KVM_F32, kb.KVM_BUDGET_FIXED, 100, 0.0, None, 0, 1e-5, 1e-12)\n"
        "assert kvm.load_library().kvm_state_rows_for(ctypes.byref(c), 64 * 9) == 100\n"
        "torch.cuda.current_device = lambda: 3\n"
        "torch.cuda.current_stream = lambda index: type('S', (), dict(cuda_stream=40 + index))\n"
        "kb._current_device = torch.cuda.current_device\n"
        "assert kb._stream() == 43\n")
    r = subprocess.run([sys.executable, "-c", program], cwd=root, capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stderr[-2000:]
