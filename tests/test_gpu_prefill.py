"""The prompt taken in whole (chunks as large as the workspace allows) against the same prompt in steps of the context's
own row capacity."""
import pytest
import torch

import workloads as wl
from workloads.device import UploadingWeights, make_context

pytestmark = pytest.mark.gpu


def _logits(ctx, w, S):
    rows = (torch.arange(w.N, device="cuda", dtype=torch.int32) * 37 % w.model.vocab).view(w.N, 1)
    out = torch.empty((w.N, 1, w.model.vocab), dtype=torch.float32, device="cuda")
    ctx.step(rows, S, torch.zeros(w.N, dtype=torch.int32, device="cuda"), logits_out=out)
    torch.cuda.synchronize()
    return out


@pytest.mark.parametrize("dtype", ["bf16", "bf16w8"])
@pytest.mark.parametrize("parts", [(1,), (33,), (129, 640), (2300, 5, 200)])
def test_whole_prompt_equals_small_steps(parts, dtype):
    """Prompts within one chunk, of one ragged row tile, appended to a cache, and past the 2048 rows of a chunk.  The
    keys and values are rounded to bfloat16 from sums in another order: a few move by one unit in the last place
    (2^-8), which leaves the next token's logits within 4e-3 of their norm."""
    S = sum(parts)
    w = wl.get_workload("c3").scaled(n_layers=2, d_model=256, n_heads=4, head_dim=64, d_ff=704, vocab=2000, N=3, gamma=4,
                                     S=S + 3, R=0, seed=1500 + S, dtype=dtype)
    dev = UploadingWeights(w.model, w.seed, "cuda:0").upload_all()
    a, b = (make_context(w.model, dev, max_branches=3, max_rows_per_branch=4, max_shared=S + 3, max_private=1) for _ in range(2))
    toks = torch.randint(0, 2000, (S,), generator=torch.Generator().manual_seed(S)).to("cuda", torch.int32)
    pos = 0
    for n in parts:
        assert a.prefill_shared(toks[pos:pos + n], pos) == pos + n
        for lo in range(pos, pos + n, 12):
            chunk = toks[lo:min(lo + 12, pos + n)].view(1, -1)
            b.step(chunk, lo, None, flags=1)
        pos += n
    x, y = _logits(a, w, S), _logits(b, w, S)
    rel = ((x - y).norm() / y.norm()).item()
    print("relative difference", rel, flush=True)
    assert rel <= 4e-3
    with pytest.raises(Exception):
        a.prefill_shared(toks[:5] if S >= 5 else torch.zeros(5, dtype=torch.int32, device="cuda"), S)
