"""Which kernels a call launches."""
import torch


def launched(call) -> str:
    with torch.profiler.profile(activities=[torch.profiler.ProfilerActivity.CUDA]) as watch:
        call()
        torch.cuda.synchronize()
    return " ".join(e.key for e in watch.key_averages() if "kernel" in e.key)
