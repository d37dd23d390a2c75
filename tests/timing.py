"""Times of calls for the tests that compare two forms of one call (ratios only,
with room for a busy device)."""
import time

import torch


def us_per_call(call, least_us=3000.0, reps=5):
    """Smallest of `reps` mean times of enough calls in a row to last least_us."""
    call()
    torch.cuda.synchronize()
    t = time.perf_counter()
    call()
    torch.cuda.synchronize()
    k = max(1, int(least_us / max((time.perf_counter() - t) * 1e6, 1.0)))
    best = float("inf")
    for _ in range(reps):
        torch.cuda.synchronize()
        t = time.perf_counter()
        for _ in range(k):
            call()
        torch.cuda.synchronize()
        best = min(best, (time.perf_counter() - t) * 1e6 / k)
    return best
