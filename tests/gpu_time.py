"""Time of a library call on the GPU, for tests that compare two calls."""


def graph_us(torch, call, n=10, replays=7):
    """Microseconds per call: the best of several replays of n calls captured in a graph."""
    s = torch.cuda.Stream()
    with torch.cuda.stream(s):
        call()
        s.synchronize()
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g, stream=s):
            for _ in range(n):
                call()
        e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        best = float("inf")
        for _ in range(replays):
            e0.record()
            g.replay()
            e1.record()
            s.synchronize()
            best = min(best, e0.elapsed_time(e1) * 1000 / n)
    return best
