"""Which of the library's kernels a call runs, for tests that have to reach a given one."""
import re


def kernels_of(fn):
    """(names of the GPU kernels that fn() runs, with their template arguments and with the step kernels'
    variants as numbers, e.g. "k_fwd_v<float, float, 16, 2>"; fn's result)."""
    import torch
    from torch.profiler import ProfilerActivity, profile
    torch.cuda.synchronize()
    with profile(activities=[ProfilerActivity.CUDA]) as prof:
        out = fn()
        torch.cuda.synchronize()
    names = set()
    for e in prof.events():
        m = re.search(r"\bk_\w+(<[^(]*>)?", e.name.replace("(pat::(anonymous namespace)::Var)", ""))
        if m:
            names.add(m.group(0))
    return names, out


def bases(names):
    """Kernel names without template arguments."""
    return {n.split("<")[0] for n in names}
