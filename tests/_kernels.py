"""Which of the library's kernels a call runs, for tests that have to reach a given one."""
import re
import time


def _trace(fn):
    import torch
    from torch.profiler import ProfilerActivity, profile
    mark = torch.empty(64, device="cuda")
    torch.cuda.synchronize()
    with profile(activities=[ProfilerActivity.CUDA]) as prof:
        # the trace keeps what lies well inside its window: leave room around the call, and
        # frame it by kernels of torch that tell a trace that lost some
        time.sleep(0.05)
        mark.fill_(1.0)
        torch.cuda.synchronize()
        out = fn()
        torch.cuda.synchronize()
        mark.fill_(2.0)
        torch.cuda.synchronize()
        time.sleep(0.05)
    return [e.name for e in prof.events()], out


def kernels_of(fn):
    """(names of the GPU kernels that fn() runs, with their template arguments and with the step kernels'
    variants as numbers, e.g. "k_fwd_v<float, float, 16, 2>"; fn's result)."""
    for _ in range(5):
        events, out = _trace(fn)
        names = set()
        for name in events:
            m = re.search(r"\bk_\w+(<[^(]*>)?", name.replace("(pat::(anonymous namespace)::Var)", ""))
            if m:
                names.add(m.group(0))
        if sum("FillFunctor" in name for name in events) >= 2:
            return names, out
    raise RuntimeError("the trace lost its first or last kernels five times")


def bases(names):
    """Kernel names without template arguments."""
    return {n.split("<")[0] for n in names}
