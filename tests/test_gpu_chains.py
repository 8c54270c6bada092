"""The backward's chains (segments of at least 48 pairs, with the workspace)
at the sizes where their code changes, bit for bit against the fp32 oracle and
within tolerance of the definition: rounds of 40 rows of a wavefront's chain,
groups of 40 in rounds of 160 of a workgroup's, the lengths where one gives
way to the other and to pieces, rows that fill a 64-column part or not, few and
many list workgroups, and more chains than one wavefront each."""
import numpy as np
import pytest

from tests.test_gpu_split import hot_batch, run_steps

pytestmark = pytest.mark.gpu

EDGES = [40, 47, 48, 49, 79, 80, 81, 119, 120, 121, 160, 161, 509, 511, 512, 513, 519, 520, 521, 639, 640, 641,
         1023, 1024, 1025, 1599, 1600, 2047]


# the workspace has 16 list workgroups up to 125 thousand pairs or so, else 256
@pytest.mark.parametrize("filler", [3_000, 130_000])
@pytest.mark.parametrize("dim", [4, 36, 64, 100, 516])
def test_chain_lengths_at_their_edges(dim, filler):
    w, b = hot_batch(EDGES, dim, filler=filler, seed=dim + filler % 7)
    print(f"\n[d{dim}] pairs {b.num_pairs}", flush=True)
    for fused in (True, False):
        run, nsplit = run_steps(w, [b], fused)
        assert nsplit == 0
        run.release()


@pytest.mark.parametrize("dim,rows,optimizer", [(260, 900, "sgd"), (16, 3000, "rmsprop")])
def test_more_chains_than_wavefronts_for_them(dim, rows, optimizer):
    """Every row hot: chains of both kinds beyond the grid are taken in turn."""
    rng = np.random.default_rng(dim)
    lengths = rng.integers(48, 130, rows)
    lengths[rng.choice(rows, 40, replace=False)] = 700
    w, b = hot_batch(lengths, dim, rows=rows + 8, filler=100, seed=dim, optimizer=optimizer)
    print(f"\n[d{dim}] pairs {b.num_pairs}", flush=True)
    run, _ = run_steps(w, [b], True)
    run.release()
