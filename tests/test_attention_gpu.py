"""GPU parity of decode attention (through the C ABI) against the fp64 oracle.

Bar: |gpu - y| <= 4e-3 * S per output element, S = sum_j p_j |v_j| (tests/parity.py), on seeded inputs
with the ragged length mix of a decode batch; empty and one-position requests, grouped heads whose
group is not a power of two, both head sizes, and chunked as well as single-pass launches."""
import numpy as np
import pytest

from tests.gpu_common import say, to_dev, to_host
from tests.parity import check, ulp16

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def thi():
    import torch
    assert torch.cuda.is_available(), "these tests need the MI355X"
    import paper_2605_25655_amd as thi
    thi.load_library()
    return thi


def f16(a):
    return np.asarray(a, dtype=np.float16)


def make_case(seed, B, Hq, Hkv, D, S_max, lens):
    rng = np.random.Generator(np.random.Philox(key=seed))
    q = f16(rng.standard_normal((B, Hq, D)))
    k = f16(rng.standard_normal((B, Hkv, S_max, D)))
    v = f16(rng.standard_normal((B, Hkv, S_max, D)))
    # whatever lies past a request's length must not matter: poison it
    for b in range(B):
        k[b, :, lens[b]:] = np.float16(np.nan)
        v[b, :, lens[b]:] = np.float16(np.inf)
    return q, k, v


def run(thi, q, k, v, lens, scale):
    import torch
    B, Hq, D = q.shape
    _, Hkv, S_max, _ = k.shape
    ws = thi.Workspace(thi.thi_attention_workspace_bytes(B, Hq, Hkv, D, S_max), init=False)
    out = torch.full((B, Hq, D), float("nan"), dtype=torch.float16, device="cuda")
    ld = torch.from_numpy(np.ascontiguousarray(lens, dtype=np.int32)).cuda()
    qd, kd, vd = to_dev(q), to_dev(k), to_dev(v)
    thi.thi_decode_attention(qd, kd, vd, ld, scale, out, ws)
    first = to_host(out)
    out2 = torch.full((B, Hq, D), float("nan"), dtype=torch.float16, device="cuda")
    thi.thi_decode_attention(qd, kd, vd, ld, scale, out2, ws)
    assert np.array_equal(first.view(np.uint16), to_host(out2).view(np.uint16)), "not reproducible"
    return first


CASES = [
    # B, Hq, Hkv, D, S_max, lengths
    (1, 4, 4, 128, 64, [64]),
    (2, 4, 4, 128, 300, [300, 1]),
    (3, 8, 8, 128, 1000, [1000, 517, 0]),
    (4, 16, 2, 128, 777, [777, 64, 65, 3]),          # group of 8
    (2, 6, 2, 128, 500, [123, 500]),                  # group of 3: two passes, the second with one head
    (2, 8, 4, 64, 600, [600, 257]),                   # head size 64, group of 2
    (5, 4, 1, 64, 130, [130, 129, 128, 127, 1]),      # group of 4
    (40, 32, 32, 128, 200, None),                     # many workgroups: one pass per request
    (1, 8, 1, 128, 4096, [4096]),                     # one request, long: cut into chunks
    (2, 64, 8, 128, 2050, [2050, 999]),               # 70B-like heads
    (2, 8, 2, 128, 333, [333, 200]),                  # group of 4, head size 128
    (1, 24, 2, 128, 450, [450]),                      # group of 12: a pass of 8 heads and a pass of 4
    (3, 32, 8, 128, 150, [150, 17, 16]),              # Llama-3-8B-like heads, short
]


@pytest.mark.parametrize("B,Hq,Hkv,D,S_max,lens", CASES)
def test_decode_attention_matches_oracle(thi, oracle_mod, B, Hq, Hkv, D, S_max, lens):
    say(f"[case] decode attention B={B} Hq={Hq} Hkv={Hkv} D={D} S_max={S_max}")
    if lens is None:
        lens = (np.arange(B) * 37 % S_max + 1).tolist()
    lens = np.asarray(lens, dtype=np.int32)
    q, k, v = make_case(9000 + B + Hq + D + S_max, B, Hq, Hkv, D, S_max, lens)
    scale = float(np.float32(1.0 / np.sqrt(D)))
    got = run(thi, q, k, v, lens, scale)
    kc, vc = k.copy(), v.copy()
    for b in range(B):                       # the oracle never reads past the length either; keep it finite anyway
        kc[b, :, lens[b]:] = 0
        vc[b, :, lens[b]:] = 0
    y, s = oracle_mod.decode_attention(q, kc, vc, lens, scale)
    check(got.reshape(B * Hq, D), y.reshape(B * Hq, D), s.reshape(B * Hq, D) + 1e-30, "decode attention", argmax=False)
    for b in range(B):
        if lens[b] == 0:
            assert not got[b].astype(np.float32).any(), "an empty request must give zeros"


def test_sharp_softmax_selects_one_row(thi, oracle_mod):
    # a dominant key: the weights are one-hot to fp32 precision, so the output is that value row bit for bit
    rng = np.random.default_rng(7)
    B, H, D, S = 2, 4, 128, 900
    q = f16(np.full((B, H, D), 4.0))
    k = f16(rng.uniform(-0.05, 0.05, (B, H, S, D)))
    v = f16(rng.standard_normal((B, H, S, D)))
    pick = [[5, 899, 400, 64], [0, 63, 128, 700]]
    for b in range(B):
        for h in range(H):
            k[b, h, pick[b][h]] = 4.0
    got = run(thi, q, k, v, np.array([S, S]), 1.0)
    for b in range(B):
        for h in range(H):
            assert np.array_equal(got[b, h].view(np.uint16), v[b, h, pick[b][h]].view(np.uint16))


@pytest.mark.parametrize("B,Hq,Hkv", [(32, 32, 32), (32, 64, 8), (1, 64, 8)])
def test_full_size_properties_without_an_oracle(thi, B, Hq, Hkv):
    """At the benchmark's size (2048 cached positions per request, heads of 128): permuting the requests
    permutes the outputs bit for bit (requests are independent), and scaling V by a power of two scales the
    output exactly (the weights do not depend on V)."""
    import torch
    D, S = 128, 2048
    say(f"[case] attention properties B={B} Hq={Hq} Hkv={Hkv} S={S}")
    g = torch.Generator(device="cuda")
    g.manual_seed(5 + B + Hkv)
    q = torch.randn((B, Hq, D), generator=g, device="cuda", dtype=torch.float32).half()
    k = torch.randn((B, Hkv, S, D), generator=g, device="cuda", dtype=torch.float32).half()
    v = torch.randn((B, Hkv, S, D), generator=g, device="cuda", dtype=torch.float32).half()
    lens = torch.randint(1, S + 1, (B,), generator=g, device="cuda", dtype=torch.int32)
    lens[0] = S
    ws = thi.Workspace(thi.thi_attention_workspace_bytes(B, Hq, Hkv, D, S), init=False)
    scale = 1.0 / D ** 0.5

    def call(q_, k_, v_, l_):
        out = torch.full((B, Hq, D), float("nan"), dtype=torch.float16, device="cuda")
        thi.thi_decode_attention(q_, k_, v_, l_, scale, out, ws)
        torch.cuda.synchronize()
        return out

    a = call(q, k, v, lens)
    assert torch.isfinite(a.float()).all()
    perm = torch.randperm(B, generator=g, device="cuda")
    ap = call(q[perm].contiguous(), k[perm].contiguous(), v[perm].contiguous(), lens[perm].contiguous())
    assert torch.equal(a[perm].view(torch.int16), ap.view(torch.int16))
    a4 = call(q, k, (v.float() * 4).half(), lens)
    ok = a.float().abs() >= 2.0 ** -12
    assert ok.float().mean() > 0.95
    assert torch.equal((a.float() * 4)[ok], a4.float()[ok])


def test_attention_argument_errors(thi):
    import torch
    z = lambda *sh: torch.zeros(sh, dtype=torch.float16, device="cuda")
    ws = thi.Workspace(1 << 20, init=False)
    lens = torch.ones(1, dtype=torch.int32, device="cuda")
    assert thi.thi_decode_attention(z(1, 3, 128), z(1, 2, 8, 128), z(1, 2, 8, 128), lens, 1.0, z(1, 3, 128), ws, check=False) == 2
    assert thi.thi_decode_attention(z(1, 2, 96), z(1, 2, 8, 96), z(1, 2, 8, 96), lens, 1.0, z(1, 2, 96), ws, check=False) == 2
    assert thi.thi_decode_attention(z(1, 2, 128), z(1, 2, 8, 128), z(1, 2, 8, 128), None, 1.0, z(1, 2, 128), ws, check=False) == 1
    assert thi.thi_attention_workspace_bytes(1, 3, 2, 128, 8) == 0


# A request is cut by its own length, and groups of four and more heads of 128 take up to 16 heads a pass: sizes around the
# 16-position blocks, the 64-position chunk grid, the 128-position minimum, the 512 positions up to which many requests stay
# whole, the 32 chunks a request may have, passes of 16 heads and a rest, more than 64 requests, and one long request among short ones.
CHUNKS = [
    (6, 8, 1, 128, 4100, [4100, 1, 0, 129, 128, 64]),
    (1, 5, 1, 128, 8192, [8192]),                     # 32 chunks
    (1, 1, 1, 64, 8191, [8191]),
    (3, 17, 1, 128, 300, [15, 16, 17]),               # a pass of 16 heads and a pass of one
    (2, 40, 2, 128, 700, [700, 193]),                 # groups of 20
    (100, 4, 1, 128, 150, None),                      # more requests than lanes, cut
    (70, 2, 1, 64, 400, None),
    (4, 64, 8, 128, 1025, [1025, 1024, 1023, 2]),
    (2, 52, 52, 128, 900, [900, 31]),
    (33, 32, 8, 128, 161, None),                      # not cut
    (32, 28, 4, 128, 700, [511, 512, 513, 700] + [97 * i % 701 for i in range(28)]),   # cut above 512 positions only
    (9, 16, 16, 128, 513, [513, 512, 1, 0, 129, 128, 511, 300, 513]),
]


@pytest.mark.parametrize("B,Hq,Hkv,D,S_max,lens", CHUNKS)
def test_chunks_of_live_lengths(thi, oracle_mod, B, Hq, Hkv, D, S_max, lens):
    """Against the oracle, and: a request's result does not depend on its place in the batch, bit for bit."""
    say(f"[case] attention chunks B={B} Hq={Hq} Hkv={Hkv} D={D} S_max={S_max}")
    if lens is None:
        lens = (np.arange(B) * 41 % (S_max + 1)).tolist()
    lens = np.asarray(lens, dtype=np.int32)
    q, k, v = make_case(9500 + B + Hq + D + S_max, B, Hq, Hkv, D, S_max, lens)
    scale = float(np.float32(1.0 / np.sqrt(D)))
    got = run(thi, q, k, v, lens, scale)
    kc, vc = np.nan_to_num(k, posinf=0.0), np.nan_to_num(v, posinf=0.0)
    y, s = oracle_mod.decode_attention(q, kc, vc, lens, scale)
    check(got.reshape(B * Hq, D), y.reshape(B * Hq, D), s.reshape(B * Hq, D) + 1e-30, "attention chunks", argmax=False)
    perm = np.random.default_rng(B).permutation(B)
    again = run(thi, q[perm], k[perm], v[perm], lens[perm], scale)
    assert np.array_equal(got[perm].view(np.uint16), again.view(np.uint16))


@pytest.mark.parametrize("B,Hq,Hkv,D,S_max", [(5, 64, 8, 128, 3000), (4, 16, 16, 128, 2000), (3, 8, 4, 64, 1500), (70, 2, 1, 64, 900), (40, 28, 4, 128, 400)])
def test_a_request_does_not_see_its_neighbours_or_the_cache_size(thi, B, Hq, Hkv, D, S_max):
    """Requests are cut into chunks; a request's bits stay the same when the other requests grow or shrink and when its
    keys and values lie in a larger cache."""
    say(f"[case] attention neighbours B={B} Hq={Hq} Hkv={Hkv} D={D} S_max={S_max}")
    rng = np.random.default_rng(B + S_max)
    L0 = S_max - 123
    full = np.full(B, S_max, dtype=np.int32)
    q, k, v = make_case(9700 + B + D, B, Hq, Hkv, D, S_max, full)
    scale = float(np.float32(1.0 / np.sqrt(D)))
    first = None
    for lens in (full.copy(), np.ones(B, np.int32), rng.integers(0, S_max + 1, B).astype(np.int32), np.zeros(B, np.int32)):
        lens[0] = L0
        got = run(thi, q, k, v, lens, scale)[0]
        first = got if first is None else first
        assert np.array_equal(got.view(np.uint16), first.view(np.uint16)), lens[:8]
    wide = np.zeros((2, B, Hkv, 2 * S_max + 77, D), np.float16)
    wide[0, :, :, :S_max], wide[1, :, :, :S_max] = k, v
    lens = np.ones(B, np.int32)
    lens[0] = L0
    got = run(thi, q, wide[0], wide[1], lens, scale)[0]
    assert np.array_equal(got.view(np.uint16), first.view(np.uint16))


@pytest.mark.parametrize("Hq,Hkv,D", [(16, 1, 128), (12, 3, 128), (4, 4, 128), (8, 2, 64)])
@pytest.mark.parametrize("L", [2, 37, 300])
def test_weights_keep_their_precision_where_values_cancel(thi, oracle_mod, Hq, Hkv, D, L):
    """Nearly equal scores and values of alternating sign: the result is what is left of the weights' differences.  Bound: the
    one rounding of the result, and 2^-17 of the sum of magnitudes for the fp32 scores (up to 16 x a few 2^-24) and weights."""
    say(f"[case] attention cancellation Hq={Hq} Hkv={Hkv} D={D} L={L}")
    rng = np.random.Generator(np.random.Philox(key=9900 + Hq + D + L))
    q = f16(rng.standard_normal((1, Hq, D)))
    k = f16(rng.standard_normal((1, Hkv, 1, D)) + 0.02 * rng.standard_normal((1, Hkv, L, D)))
    sign = np.where(np.arange(L) % 2 == 0, 1.0, -1.0)[None, None, :, None]
    v = f16(sign * np.ones((1, Hkv, L, D)))
    lens = np.array([L], np.int32)
    scale = float(np.float32(1.0 / np.sqrt(D)))
    got = run(thi, q, k, v, lens, scale).astype(np.float64)
    y, s = oracle_mod.decode_attention(q, k, v, lens, scale)
    err = np.abs(got - y)
    assert (err <= 0.5 * ulp16(y) + 2.0 ** -17 * s).all(), float((err / s).max())
    # an infinite value stands for itself in its own column and nowhere else
    v[0, :, L // 2, 3], v[0, :, 0, 5] = np.inf, -np.inf
    got = run(thi, q, k, v, lens, scale).astype(np.float64)
    assert (got[..., 3] == np.inf).all() and (got[..., 5] == -np.inf).all()
    keep = np.delete(np.arange(D), [3, 5])
    assert (np.abs(got - y) <= 0.5 * ulp16(y) + 2.0 ** -17 * s)[..., keep].all()


@pytest.mark.parametrize("Hq,Hkv,D", [(64, 8, 128), (8, 8, 64)])
def test_attention_replays_from_a_captured_graph(thi, Hq, Hkv, D):
    """One captured call, replayed with other lengths and queries than it was captured with (the chunks are chosen from the lengths on
    the device), eager calls and synchronisations in between: every replay equals the eager call bit for bit."""
    import torch
    B, S = 3, 1500
    say(f"[case] attention graph Hq={Hq} Hkv={Hkv} D={D}")
    gen = torch.Generator(device="cuda")
    gen.manual_seed(77 + D)
    q, k, v = (torch.empty(s, dtype=torch.float16, device="cuda").normal_(generator=gen)
               for s in ((B, Hq, D), (B, Hkv, S, D), (B, Hkv, S, D)))
    lens = torch.tensor([S, 700, 1], dtype=torch.int32, device="cuda")
    out = torch.full((B, Hq, D), float("nan"), dtype=torch.float16, device="cuda")
    ws = thi.Workspace(thi.thi_attention_workspace_bytes(B, Hq, Hkv, D, S), init=False)
    stream, graph = torch.cuda.Stream(), torch.cuda.CUDAGraph()
    with torch.cuda.stream(stream):
        thi.thi_decode_attention(q, k, v, lens, D ** -0.5, out, ws)
        stream.synchronize()
        with torch.cuda.graph(graph, stream=stream):
            thi.thi_decode_attention(q, k, v, lens, D ** -0.5, out, ws)
    torch.cuda.synchronize()
    for new in ([1, S, 0], [129, 128, 127], [S, S, S], [64, 900, 1499]):
        lens.copy_(torch.tensor(new, dtype=torch.int32))
        q.normal_(generator=gen)
        thi.thi_decode_attention(q, k, v, lens, D ** -0.5, out, ws)
        torch.cuda.synchronize()
        eager = out.clone()
        out.fill_(float("nan"))
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(out.view(torch.int16), eager.view(torch.int16)), new
