"""Steps on carried pair sums captured into a HIP graph on the stream that produced the sums: a replay starts
where the captured steps started, so what they read has to be what the last replay, or any eager step
in between, left."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("before,captured,between", [(1, 1, 1), (2, 1, 2), (1, 2, 1), (2, 3, 1), (0, 1, 1), (0, 2, 3)])
@pytest.mark.parametrize("n,D", [(8, 20_001), (12, 5_001), (16, 8_577), (24, 5_000), (24, 80_001), (32, 8_577), (32, 20_001), (40, 5_001)])
def test_carried_steps_replayed_between_eager_ones(n, D, before, captured, between):
    from paper_2306_06528_amd import svgd
    g = torch.Generator().manual_seed(n + D)
    X = (0.3 * torch.randn(n, D, generator=g)).cuda()
    G = torch.randn(n, D, generator=g).cuda()
    eps = 0.05
    Y, PHI = X.clone(), torch.empty_like(X)
    torch.cuda.synchronize()
    side = torch.cuda.Stream()
    with svgd.Svgd(n, D) as plain, svgd.Svgd(n, D, flags=svgd.FLAG_CARRY_GRAM) as eng, torch.cuda.stream(side):
        def check(steps, what):
            """X is where `steps` plain steps from Y lead, and the last of them used the h of its X."""
            for _ in range(steps):
                h_ref = plain.bandwidth(Y)
                plain.step(Y, G, eps)
            torch.cuda.synchronize()
            h, _ = eng.get_last(n)
            assert abs(h - h_ref) <= 1e-6 * h_ref, f"{what}: h {h}, of the particles {h_ref}"
            assert float((X - Y).abs().max()) <= 4e-7 * float(Y.abs().max()), what

        def eager(steps, what):
            for k in range(steps):
                eng.step(X, G, eps)
                check(1, f"{what}, step {k}")

        eager(before, "before the capture")
        torch.cuda.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=side):
            for _ in range(captured):
                eng.step(X, G, eps)
        if before:
            eager(1, "between capture and replay")
        for k in range(3):
            graph.replay()
            check(captured, f"replay {k}")
        eager(between, "after three replays")
        for k in range(2):
            graph.replay()
            check(captured, f"replay {k} after eager steps")
        # sums that are recomputed in between, by calls that use the scratch for themselves
        eng.phi(X, G, PHI)
        graph.replay()
        check(captured, "replay after svgd_phi")
        eng.bandwidth(X)
        eager(1, "after svgd_bandwidth")
        graph.replay()
        check(captured, "replay after recomputed sums")
        Y.copy_(X)
        torch.cuda.synchronize()
