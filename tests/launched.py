"""Names of the GPU kernels that a call launches, for tests of which kernel a shape takes."""
import torch


def kernels_of(call):
    """`call` runs once before (code loading, allocations) and once under the profiler."""
    call()
    torch.cuda.synchronize()
    with torch.profiler.profile(activities=[torch.profiler.ProfilerActivity.CUDA]) as prof:
        call()
        torch.cuda.synchronize()
    return [e.name for e in prof.events() if e.device_type == torch.autograd.DeviceType.CUDA and not e.name.startswith("Mem")]
