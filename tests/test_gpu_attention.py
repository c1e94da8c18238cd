"""FlowKV decode attention (q4nx_flowkv_decode) against the float64 oracle.

Tolerance per output element: |o - o_ref| <= 2e-3 * sum_j p_j |v_j| + 1e-6
(plus half a bf16 ulp of o_ref for bf16 outputs).  Scores are float32 sums of
exact bf16 products (relative error below d * 2^-24 of sum |q k|); the
weighted sums run over up to 2^15 positions in float32 (below L * 2^-24
relative to sum p |v| in the worst case, far less in practice); the chunk
merge adds a few roundings more.
"""
import numpy as np
import pytest

import oracle
from oracle.attention import decode_attention, attended_range

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def q4():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2602_06063_amd as mod
    return mod


def _case(H, G, d, L, seed):
    rng = np.random.default_rng(seed)
    q = oracle.f32_to_bf16(rng.standard_normal((H, d), dtype=np.float32))
    K = oracle.f32_to_bf16(rng.standard_normal((G, L, d), dtype=np.float32))
    V = oracle.f32_to_bf16(rng.standard_normal((G, L, d), dtype=np.float32))
    return q, K, V


def _dev(bits):
    return torch.from_numpy(np.ascontiguousarray(bits).view(np.int16)).cuda()


CASES = [
    # (H, G, d, L, t, window)  -- Gemma3 1B (4 heads, 1 group, d 256), 4B (8, 4, 256), 27B (32, 16, 128)
    (8, 4, 256, 4096, 0, 0),
    (8, 4, 256, 4096, 255, 0),
    (8, 4, 256, 4096, 256, 0),
    (8, 4, 256, 4096, 1000, 0),
    (8, 4, 256, 4096, 4095, 0),
    (8, 4, 256, 4096, 4095, 1024),
    (8, 4, 256, 4096, 700, 1024),
    (8, 4, 256, 4096, 2000, 1),
    (4, 1, 256, 2048, 1500, 0),
    (32, 16, 128, 4096, 3000, 0),
    (32, 16, 128, 4096, 3000, 1024),
    (8, 1, 64, 1024, 777, 0),
    (8, 4, 256, 32768, 32767, 0),
    # 1B geometry at 30K: 469 chunks of 64, more than a merge slice holds in
    # registers (the two-pass merge)
    (4, 1, 256, 32768, 30000, 0),
    (32, 16, 128, 32768, 20000, 0),
    # sliding windows of 1000 positions (a ragged last chunk: 40 positions
    # of a 64-position chunk, or 8 of a 32-position one) with at least 64
    # chunk workgroups: K and V requested with the query
    (32, 16, 128, 4096, 1500, 1000),
    (64, 16, 64, 2048, 1500, 1000),
    (8, 4, 256, 4096, 3000, 1000),
    # grids of 64-position chunks below one workgroup per CU take 32-position
    # chunks (K and V requested with the query from 64 workgroups): d = 128
    # and d = 64, whole and ragged last chunks
    (16, 4, 128, 2048, 1023, 1024),
    (16, 8, 64, 2048, 2000, 1000),
    # one KV group: 16-position chunks, with K and V requested early (64
    # chunks) and without (63, a ragged last chunk of 8), d = 256 and 128
    (4, 1, 256, 2048, 2047, 1024),
    (4, 1, 256, 2048, 1500, 1000),
    (8, 1, 128, 4096, 3000, 1024),
    # many heads: the merge takes 64, 128 and 256 dims per workgroup
    (64, 16, 128, 2048, 1999, 0),
    (128, 16, 128, 1024, 900, 0),
    (128, 16, 256, 1024, 1000, 0),
]


@pytest.mark.parametrize("H,G,d,L,t,window", CASES)
def test_flowkv_decode_vs_oracle(q4, H, G, d, L, t, window):
    print("[case] flowkv", H, G, d, L, t, window, flush=True)
    q, K, V = _case(H, G, d, L, seed=H * 1000 + t)
    scale = 1.0 / np.sqrt(d)
    j0, j1 = attended_range(t, window)
    work = torch.empty(q4.q4nx_flowkv_workspace_size(H, d, j1 - j0) // 4, dtype=torch.float32, device="cuda")
    o = torch.full((H, d), float("nan"), dtype=torch.float32, device="cuda")
    q4.q4nx_flowkv_decode(_dev(q), _dev(K), _dev(V), H, G, d, L, t, window, float(scale), o, work)
    torch.cuda.synchronize()
    ref, bound = decode_attention(q, K, V, t, window, scale)
    got = o.cpu().numpy().astype(np.float64)
    err = np.abs(got - ref)
    tol = 2e-3 * bound + 1e-6
    assert (err <= tol).all(), float((err / tol).max())


def test_flowkv_bf16_output_and_repeatable(q4):
    H, G, d, L, t = 8, 4, 256, 4096, 3333
    q, K, V = _case(H, G, d, L, seed=5)
    scale = 1.0 / 16.0
    work = torch.empty(q4.q4nx_flowkv_workspace_size(H, d, t + 1) // 4, dtype=torch.float32, device="cuda")
    o = torch.empty((H, d), dtype=torch.bfloat16, device="cuda")
    qd, Kd, Vd = _dev(q), _dev(K), _dev(V)
    q4.q4nx_flowkv_decode(qd, Kd, Vd, H, G, d, L, t, 0, scale, o, work)
    first = o.clone()
    q4.q4nx_flowkv_decode(qd, Kd, Vd, H, G, d, L, t, 0, scale, o, work)
    torch.cuda.synchronize()
    assert torch.equal(first.view(torch.int16), o.view(torch.int16))
    ref, bound = decode_attention(q, K, V, t, 0, scale)
    got = o.float().cpu().numpy().astype(np.float64)
    assert (np.abs(got - ref) <= 2e-3 * bound + 1e-6 + 2.0 ** -8 * np.abs(ref)).all()


# The edges of phase 1's split: one wave per workgroup with one, a whole and a
# ragged sub-chunk (16 positions for d = 256 and 128, 32 for 64), the last
# shapes of one, two and four such waves per workgroup (128, 256 and 512
# sub-chunks) and the first of the next kind, chunks of even rounds (waves with
# no position in the last chunk, one position in the last chunk, more than one
# round), and every number of query heads per group at every d.
@pytest.mark.parametrize("H,G,d,n", [(8, 4, 256, 16), (8, 4, 256, 17), (32, 16, 128, 31), (8, 8, 64, 65),
                                     (8, 4, 256, 2048), (8, 4, 256, 2049), (16, 16, 128, 1024), (16, 16, 128, 1025),
                                     (4, 1, 256, 8193), (8, 1, 256, 900), (8, 1, 128, 20000), (64, 8, 256, 4100),
                                     (64, 8, 64, 4100), (4, 1, 256, 2049), (4, 1, 256, 4097), (8, 1, 256, 4096),
                                     (2, 1, 128, 4000), (1, 1, 64, 8200), (4, 1, 64, 4097), (2, 1, 64, 33),
                                     (16, 8, 256, 9000), (16, 16, 128, 16385), (4, 1, 128, 70000), (2, 2, 64, 140001)])
def test_flowkv_split_edges(q4, H, G, d, n):
    print("[case] flowkv split", H, G, d, n, flush=True)
    q, K, V = _case(H, G, d, n + 3, seed=n)
    scale = 1.0 / np.sqrt(d)
    work = torch.full((q4.q4nx_flowkv_workspace_size(H, d, n) // 4,), float("nan"), dtype=torch.float32, device="cuda")
    o = torch.full((H, d), float("nan"), dtype=torch.float32, device="cuda")
    q4.q4nx_flowkv_decode(_dev(q), _dev(K), _dev(V), H, G, d, n + 3, n - 1, 0, float(scale), o, work)
    torch.cuda.synchronize()
    ref, bound = decode_attention(q, K, V, n - 1, 0, scale)
    assert (np.abs(o.cpu().numpy().astype(np.float64) - ref) <= 2e-3 * bound + 1e-6).all()


# Ranges that end inside a sub-chunk, one wave and four waves per workgroup:
# the lanes past the end must not weigh the last row again, where 0 times an
# infinity would be NaN.
@pytest.mark.parametrize("H,G,d,n", [(8, 4, 256, 17), (8, 8, 64, 70), (16, 4, 128, 2500)])
def test_flowkv_infinite_last_value(q4, H, G, d, n):
    print("[case] flowkv infinite value", H, G, d, n, flush=True)
    q, K, V = _case(H, G, d, n, seed=d)
    V[:, n - 1, 3], V[:, n - 1, 5] = 0x7F80, 0xFF80  # +inf, -inf
    scale = 1.0 / np.sqrt(d)
    work = torch.full((q4.q4nx_flowkv_workspace_size(H, d, n) // 4,), float("nan"), dtype=torch.float32, device="cuda")
    o = torch.empty((H, d), dtype=torch.float32, device="cuda")
    q4.q4nx_flowkv_decode(_dev(q), _dev(K), _dev(V), H, G, d, n, n - 1, 0, float(scale), o, work)
    got = o.cpu().numpy().astype(np.float64)
    assert (got[:, 3] == np.inf).all() and (got[:, 5] == -np.inf).all()
    V[:, n - 1, 3] = V[:, n - 1, 5] = 0
    ref, bound = decode_attention(q, K, V, n - 1, 0, scale)
    rest = np.delete(np.arange(d), [3, 5])
    assert (np.abs(got - ref)[:, rest] <= 2e-3 * bound[:, rest] + 1e-6).all()


@pytest.mark.parametrize("H,G,d,n", [(8, 1, 256, 2016 * 512), (64, 16, 128, 496 * 512)])
def test_flowkv_static_serves_its_longest_ranges(q4, H, G, d, n):
    """The static scratch holds as many chunks of 512 positions as its 16 MiB
    allow (2016 of 8 heads at d = 256): such a range, where shorter chunks
    would not fit, is accepted, with the bits of the workspace call."""
    print("[case] flowkv static limit", H, G, d, n, flush=True)
    g = torch.Generator(device="cuda").manual_seed(n)
    q = torch.randn(H, d, device="cuda", generator=g).bfloat16()
    K = torch.randn(G, n, d, device="cuda", generator=g, dtype=torch.bfloat16)
    V = torch.randn(G, n, d, device="cuda", generator=g, dtype=torch.bfloat16)
    work = torch.empty(q4.q4nx_flowkv_workspace_size(H, d, n) // 4, dtype=torch.float32, device="cuda")
    o = [torch.full((H, d), float("nan"), device="cuda") for _ in range(2)]
    q4.q4nx_flowkv_decode(q, K, V, H, G, d, n, n - 1, 0, 0.05, o[0], work)
    q4.q4nx_flowkv_decode_static(q, K, V, H, G, d, n, n - 1, 0, 0.05, o[1])
    torch.cuda.synchronize()
    assert torch.isfinite(o[0]).all() and torch.equal(o[0].view(torch.int32), o[1].view(torch.int32))
    p = torch.softmax(0.05 * (K[0].float() @ q[:H // G].float().T), dim=0)      # group 0, float32
    assert torch.allclose(p.T @ V[0].float(), o[0][:H // G], rtol=0, atol=1e-3)
