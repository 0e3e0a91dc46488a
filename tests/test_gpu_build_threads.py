"""Builds of different sizes from several threads at once: the subtree kernel's
LDS limit is shared by all of them.  Every tree equals the one built alone."""
import threading

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d", [3, 8, 16, 32])
def test_builds_of_many_sizes_at_once(d):
    import torch
    from paper_1304_4327_amd import knn
    rng = np.random.default_rng(d)
    sizes = [7000, 60, 3900, 900, 20_000, 1500]
    sets = [torch.from_numpy(rng.standard_normal((n, d)).astype(np.float32)).cuda() for n in sizes]
    torch.cuda.synchronize()

    def arrays(tree):
        return {k: v for k, v in knn.tree_arrays(tree).items() if isinstance(v, np.ndarray)}

    alone = []
    for x in sets:
        t = knn.knn_build_tree(x, 32)
        alone.append(arrays(t))
        t.close()
    wrong = []

    def work(first):
        try:
            s = torch.cuda.Stream()
            for i in range(12):
                j = (first + i) % len(sets)
                t = knn.knn_build_tree(sets[j], 32, stream=s)
                got = arrays(t)
                t.close()
                if any(not np.array_equal(got[k], alone[j][k]) for k in alone[j]):
                    wrong.append((first, i, sizes[j]))
        except Exception as e:  # pragma: no cover
            wrong.append((first, repr(e)))

    threads = [threading.Thread(target=work, args=(f,)) for f in range(4)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    print(f"threads d={d}: {wrong}", flush=True)
    assert not wrong
