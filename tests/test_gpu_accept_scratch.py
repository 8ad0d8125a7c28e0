"""The accept / resample step with caller-provided scratch against the entry point without, and the draw at vocabulary
sizes around its segment boundaries and from misaligned rows against the oracle."""
import ctypes as C

import numpy as np
import pytest
import torch

import oracle
import workloads as wl
from workloads.device import f32, i32

pytestmark = pytest.mark.gpu


def _inputs(N, G, V):
    rng = np.random.default_rng(N * V + G)
    z = (rng.standard_normal((N, G + 1, V)) * 2.0).astype(np.float32)
    q = oracle.softmax_temperature(z[:, :G] + rng.standard_normal((N, G, V)).astype(np.float32), 1.0)
    u = wl.uniform24(V + 3, (2, N, G))
    return z, q, wl.draw_tokens(q, u[0]), u[1], wl.uniform24(V + 4, (N,))


@pytest.mark.parametrize("V", [4, 36, 2044, 2046, 2048, 32764, 32768, 32772])
def test_draw_at_segment_edges_is_bit_exact(V):
    """PROBS mode with bonus rows: residual and plain draws."""
    import paper_2406_18200_amd as sv
    z, q, drafts, u_acc, u_res = _inputs(5, 3, V)
    p = oracle.softmax_temperature(z, 1.0)
    want = oracle.accept_resample(p, q, drafts, u_acc, u_res)
    got = sv.accept_resample(f32(p), f32(q), i32(drafts), f32(u_acc), f32(u_res), kind="probs")
    for w, g in zip(want, got):
        assert np.array_equal(w, g.cpu().numpy())


def test_draw_from_rows_off_a_16_byte_boundary():
    import paper_2406_18200_amd as sv
    z, q, drafts, u_acc, u_res = _inputs(4, 2, 1000)
    p = oracle.softmax_temperature(z, 1.0)
    off = [torch.empty(x.size + 1, dtype=torch.float32, device="cuda")[1:].view(x.shape).copy_(f32(x)) for x in (p, q)]
    want = oracle.accept_resample(p, q, drafts, u_acc, u_res)
    got = sv.accept_resample(off[0], off[1], i32(drafts), f32(u_acc), f32(u_res), kind="probs")
    for w, g in zip(want, got):
        assert np.array_equal(w, g.cpu().numpy())


@pytest.mark.parametrize("N,G,V", [(1, 1, 16), (16, 6, 32000), (40, 3, 4100), (3, 4, 40000)])
def test_scratch_form_against_the_one_without(N, G, V):
    """LOGITS mode: the statistics are summed in another order, so p(x) agrees to a few float32 roundings (4 x 2^-24 per
    combining step, 1e-6) and tokens agree (no accept test or draw of these seeds lies that close to its threshold)."""
    import paper_2406_18200_amd as sv
    from paper_2406_18200_amd import binding as B
    z, q, drafts, u_acc, u_res = (x for x in _inputs(N, G, V))
    args = [f32(z), f32(q), i32(drafts), f32(u_acc), f32(u_res)]
    got = sv.accept_resample(*args, kind="logits", temperature=0.8)
    outs = B._accept_outputs(N, G, "cuda")
    a = B._accept_struct(N, G, G + 1, V, B.SEED_KIND_LOGITS, False, 0.8, *args, *outs, None)
    lib = sv.load_library()
    B._check(lib.seed_accept_resample(C.byref(a), B._stream_handle()))
    for g, w in zip(got[:3], outs[:3]):
        assert torch.equal(g, w)
    assert ((got[3] - outs[3]).abs() <= 1e-6 * outs[3].abs()).all()
    need = lib.seed_accept_scratch_bytes(N, G + 1)
    buf = torch.empty(need, dtype=torch.uint8, device="cuda")
    assert lib.seed_accept_resample_ws(C.byref(a), B._ptr(buf), need - 1, B._stream_handle()) == -3
    assert lib.seed_accept_resample_ws(C.byref(a), None, need, B._stream_handle()) == -4
