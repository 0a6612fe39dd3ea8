"""Which kernels a call launches, by the profiler that comes with torch."""
import torch
from torch.profiler import ProfilerActivity, profile


def launched(call):
    """call()'s result and the names of the kernels it launched"""
    torch.cuda.synchronize()
    with profile(activities=[ProfilerActivity.CUDA], acc_events=True) as p:
        result = call()
        torch.cuda.synchronize()
    return result, [e.name for e in p.events() if e.device_type == torch.autograd.DeviceType.CUDA]
