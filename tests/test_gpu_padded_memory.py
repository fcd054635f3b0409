"""The padded propagation holds its input and its output, and no third array."""
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_fft", [60, 62, 128])  # an FFT of N points, the dense passes, a padded FFT
def test_no_third_array(gpu_lib, n_fft):
    n = 60
    w = torch.zeros((n,) * 4, dtype=torch.complex64, device="cuda")
    size = w.numel() * w.element_size()
    torch.cuda.synchronize()
    base = torch.cuda.memory_allocated()
    torch.cuda.reset_peak_memory_stats()
    out, _ = gpu_lib.propagate_padded(w, 20e-6, 633e-9, 0.3, n_fft)
    torch.cuda.synchronize()
    assert torch.cuda.max_memory_allocated() - base < 1.5 * size
    del out
    torch.cuda.reset_peak_memory_stats()
    gpu_lib.propagate_padded(w, 20e-6, 633e-9, 0.3, n_fft, out=w)
    torch.cuda.synchronize()
    assert torch.cuda.max_memory_allocated() - base < 0.5 * size
