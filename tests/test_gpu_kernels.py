"""GPU parity of single kernels at the sizes where their tiling, splits and dispatch can go
wrong: edges of tiles, remainders, and the smallest and largest work of a path, against the
CPU oracle within the scaled-error bound of tests/_util.py."""
import numpy as np
import pytest
import torch

import ttgen
from tests._util import abs_case, assert_close

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def lib():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2609_03459_amd as P

    return P


def _check(lib, orc, case, name, backward=True, **kw):
    """Forward (and backward) of `case` against the oracle, every element."""
    print(f"[{name}] T={case['T']} n={case['n']} d={case['d']} R={case['R']} B={case['B']} M={case['idx'].size}",
          flush=True)
    G = [torch.from_numpy(np.ascontiguousarray(case[k])).cuda() for k in ("G1", "G2", "G3")]
    idx = torch.from_numpy(np.ascontiguousarray(case["idx"], dtype=np.int64)).cuda()
    off = None if case["offsets"] is None else torch.from_numpy(np.ascontiguousarray(case["offsets"])).cuda()
    emb = lib.TTEmbedding(case["T"], case["N"], case["n"], case["d"], case["R"], max_indices=max(idx.numel(), 1),
                          max_bags=max(int(case["B"]), 1), **kw)
    out = emb.forward(*G, idx, off, num_bags=case["B"])
    V = out.cpu().numpy().reshape(case["T"] * case["B"], -1)
    assert emb.check_errors() == 0
    assert_close(f"forward {name}", V, orc.forward(case)[0], orc.forward(abs_case(case))[0])
    if not backward:
        return emb
    dV = torch.from_numpy(np.ascontiguousarray(case["dV"])).cuda()
    grads = emb.backward(*G, idx, off, dV, num_bags=case["B"], reuse_grouping=True)
    torch.cuda.synchronize()
    ref, mag = orc.backward(case)[:3], orc.backward(abs_case(case))[:3]
    for k in range(3):
        assert_close(f"dG{k + 1} {name}", grads[k].cpu().numpy(), ref[k], mag[k])
    return emb


@pytest.mark.parametrize("runs", [1, 7, 8 * 384 - 1, 8 * 384, 8 * 384 + 9])
def test_chunks_by_rank_and_by_claim(lib, orc, runs):
    # every (table, i2) run is one chunk here: fewer chunks than queues, than workers (on 256
    # CUs the R = 32 forward has 3,072, 384 in each of eight queues, and the backward 1,024 per
    # owner), exactly as many, and a few more, so that chunks are taken by rank, claimed and stolen
    case = ttgen.tiny(8100 + runs % 97, 1, (2, runs, 2), (4, 4, 8), 32, B=3 * runs, single=True)
    _check(lib, orc, case, f"{runs} chunks")
