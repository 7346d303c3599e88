"""The GPU kernels that a call launches, by name, for bounds from above: torch's
profiler sees every kernel of the process, but may lose the record of one."""
import torch
from torch.profiler import ProfilerActivity, profile


def launched(call):
    """Names of the kernels of call(), the library's without their namespace."""
    torch.cuda.synchronize()
    with profile(activities=[ProfilerActivity.CUDA]) as p:
        call()
        torch.cuda.synchronize()
    names = [e.name for e in p.events() if e.device_type == torch.autograd.DeviceType.CUDA]
    return [n.split("(anonymous namespace)::", 1)[-1] for n in names if not n.startswith(("Memcpy", "Memset"))]


def count(names, kernel):
    """Launches of one kernel of the library, whatever its template arguments."""
    return sum(n.startswith((kernel + "<", kernel + "(")) for n in names)
