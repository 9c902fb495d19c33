"""The autotuner times the automatic choice among its candidates, so that a recorded
entry is not slower than none: depths of 13 and 14 are chosen, but tried of one shape only."""
import pytest

torch = pytest.importorskip("torch")
pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not torch.cuda.is_available(), reason="needs a GPU")]


@pytest.mark.parametrize("m,n,iters", [(400, 400, 14), (500, 500, 14), (560, 560, 13), (64, 64, 100), (700, 700, 1),
                                       (900, 900, 20)])
def test_the_automatic_choice_is_a_candidate(m, n, iters):
    import paper_2109_05496_amd as ctv
    ctv.tune_cache_clear()
    b = torch.view_as_complex(torch.randn(m, n, 2, device="cuda")).contiguous()
    T, _, waves, rows = ctv.tiling(0, iters, m, n, detail=True)
    try:
        for _ in range(2):  # the second time with an entry recorded
            r = ctv.autotune(b, 0.05, iters=iters, reps=1)
            tried = [(c["fuse"], c["tile"]) for c in r["candidates"]]
            assert tried.count((T, (waves, rows))) == 1 and len(set(tried)) == len(tried) <= 63
            assert r["best"] in r["candidates"]
    finally:
        ctv.tune_cache_clear()
