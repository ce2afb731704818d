"""What the binding allocates, when there is no memory for it."""
import pytest
import torch

import paper_2509_07103_amd as pkg

pytestmark = pytest.mark.gpu


@pytest.fixture
def little_memory():
    """256 MiB beyond what the process holds (a limit of torch's allocator: the device is not asked)."""
    dev = torch.device("cuda:0")
    pkg.lib()
    torch.cuda.empty_cache()
    total = torch.cuda.get_device_properties(dev).total_memory
    torch.cuda.set_per_process_memory_fraction((torch.cuda.memory_reserved(dev) + (256 << 20)) / total, dev)
    yield dev
    torch.cuda.set_per_process_memory_fraction(1.0, dev)
    torch.cuda.empty_cache()


@pytest.mark.parametrize("what", ["output", "workspace", "packed"])
def test_no_memory_is_torch_out_of_memory_error(little_memory, what):
    """Callers catch torch.OutOfMemoryError to go on with a smaller batch, and the next call works."""
    dev = little_memory
    if what == "output":            # 1 GiB of y
        desc = pkg.LayerDesc(2, 4096, 3)
        P, x = torch.zeros(desc.coef_shape(), device=dev), torch.zeros((1 << 16, 2), device=dev)
        call = lambda: pkg.lmkan_forward(desc, x, P)
    elif what == "workspace":       # 35 MB of inputs and 180 MiB of something else leave no room for the sorted stream
        desc = pkg.LayerDesc(64, 4, 16)
        P, gp = torch.zeros(desc.coef_shape(), device=dev), torch.zeros(desc.coef_shape(), device=dev)
        x, gy = torch.zeros((1 << 17, 64), device=dev), torch.zeros((1 << 17, 4), device=dev)
        assert pkg.lmkan_workspace_bytes(desc, 1 << 17, True, False, True) > 100 << 20
        other = torch.empty(180 << 20, dtype=torch.uint8, device=dev)
        call = lambda: pkg.lmkan_backward(desc, x, None, gy, need_grad_x=False, grad_coef=gp)
    else:                           # one output, packed: 64 columns, 1.1 GB
        desc = pkg.LayerDesc(2048, 1, 64)
        P = torch.zeros(desc.coef_shape(), device=dev)
        call = lambda: pkg.lmkan_pack(desc, P)
    with pytest.raises(torch.OutOfMemoryError):
        call()
    assert pkg.lmkan_forward(desc, torch.zeros((4, desc.n_in), device=dev), P).shape == (4, desc.n_out)
