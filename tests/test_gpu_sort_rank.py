"""The sort at the edges of its ranking launch: keys and the stable
permutation bit-exact where the runs fill one and two rounds of searches, and
on both sides of the size where merges take over."""
import pytest

from test_gpu_sort import test_sort_is_stable as check

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [8191, 9216, 9217, 12287, 12288, 12289, 13000])
@pytest.mark.parametrize("kind", ["random", "equal", "descending"])
def test_ranked_sort_is_stable(oracle, n, kind):
    print(f"sort n={n} {kind}", flush=True)
    check(oracle, n, kind)
