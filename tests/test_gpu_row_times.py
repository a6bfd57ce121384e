"""The forms of the row kernels by the time they take: few rows take no longer than rows half as long
again, which have the same number of launches and more to read, and a call just past a border of a
rule no longer than one just before it."""
import pytest

pytestmark = pytest.mark.gpu

# kind, 16-byte words of a row, rows, words of the row that it is compared with, bound
CASES = [
    ("rows", 1000, 64, 1500, 1.1),    # one wavefront per row took 1.4 times as long
    ("rows", 1000, 256, 1500, 1.1),
    ("rows", 8200, 64, 8100, 1.06),   # past the border of the pipelined form: 1.11
    ("pairs", 1000, 64, 1500, 1.1),   # one wavefront per token took 1.3 times as long
    ("pairs", 1000, 256, 1500, 1.1),  # and here 1.5 times
    ("grad", 250, 256, 400, 1.0),     # one wavefront per row took 1.06 times as long
    ("grad", 1500, 64, 2000, 1.1),    # four 1.2 times
    ("grad", 1300, 256, 2000, 1.05),  # four 1.12 times
]


def _graph(kind, words, rows):
    import torch
    import paper_2609_14636_amd as P
    V = words * 8
    t, s = (torch.empty((rows, V), dtype=torch.bfloat16, device="cuda").normal_(0, 3) for _ in range(2))
    ids = torch.randint(0, V, (rows,), dtype=torch.int32, device="cuda")
    lay = P.Layout(torch.tensor([0, 1], dtype=torch.int32, device="cuda"),
                   torch.tensor([0, rows], dtype=torch.int64, device="cuda"), rows)
    path = P.Path(lay, P.STRIDE_UNIT_TOKEN, exact_kl=kind == "pairs")
    path.score(V, [t], s, ids)
    path.stop_unit.fill_(-1)
    grad = torch.empty_like(s)

    def call():
        if kind == "grad":
            path.grad(V, s, ids, grad)
        else:
            path.score(V, [t], s, ids)
    call()
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        for _ in range(20):
            call()
    return graph, (t, s, ids, path, grad)


@pytest.mark.parametrize("kind,words,rows,other,bound", CASES)
def test_not_slower_than_a_neighbour(kind, words, rows, other, bound):
    import torch
    pair = [_graph(kind, w, rows) for w in (words, other)]
    best = [float("inf"), float("inf")]
    for rep in range(12):
        for i in (0, 1):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            pair[i][0].replay()
            a.record()
            pair[i][0].replay()
            b.record()
            torch.cuda.synchronize()
            best[i] = min(best[i], a.elapsed_time(b) * 50)
    print(f"{kind}, {rows} rows: {words} words {best[0]:.2f} us, {other} words {best[1]:.2f} us", flush=True)
    assert best[0] <= bound * best[1]
