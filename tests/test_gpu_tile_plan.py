"""The 256-query tiles of an attention call are divided between kernels by their
number: whole rounds of 256 tiles (one per compute unit) on the plain kernel, a
last round of at most 128 tiles in halves or quarters.  The small parity cases
all fall to the latter; here the plain kernel runs at the same small sizes
(129 to 256 tiles), both together (257 and more), and the counts on either
side of the line, with the options that have instantiations of their own.
Sampled heads, among them those at the border, against the oracle: S and the
running maxima bit for bit, P codes outside the tie band bit for bit, O within
2e-3 of its largest value.
"""
import numpy as np
import pytest

import pcode_check
from test_gpu_int4 import FORMATS, O_TOL, _cfg, _geo, _inputs, _params, _ra, _run_quant, _torch

pytestmark = pytest.mark.gpu

# heads, grid, case (rotation, q_group, k_group, v_group, kv_block, P mapping, smoothing, V Hadamard, l from codes)
PLANS = [
    (64, (1, 3, 5), (1, 128, 128, 128, 128, 0, 3, 0, 0)),      # 64 tiles: all in quarters
    (65, (1, 3, 5), (1, 128, 128, 128, 128, 0, 3, 0, 0)),      # 65: all in halves
    (33, (3, 10, 10), (2, 64, 32, 128, 128, 0, 7, 1, 1)),      # 66 in halves, 300 tokens, key bias
    (64, (3, 10, 10), (2, 1, 1, 128, 64, 1, 3, 0, 0)),         # 128 in halves, kv_block 64, per-token
    (128, (1, 3, 5), (1, 1, 1, 128, 128, 0, 3, 0, 0)),         # 128 per-token: quarters
    (129, (1, 3, 43), (1, 128, 64, 128, 64, 0, 7, 0, 0)),      # 129 plain, kv_block 64, key bias
    (193, (3, 10, 10), (1, 128, 128, 128, 128, 0, 3, 0, 0)),   # 386: 256 plain, then 130: plain too
    (165, (3, 10, 10), (1, 128, 128, 128, 128, 0, 3, 0, 0)),   # 330: 256 plain, 74 in halves
    (129, (1, 3, 43), (1, 128, 128, 128, 128, 0, 3, 0, 0)),    # 129: all plain, two blocks, the second of one key
    (65, (3, 10, 10), (1, 1, 1, 128, 128, 0, 7, 0, 0)),        # 130 plain, per-token scales with the key bias
    (130, (1, 8, 16), (2, 128, 32, 256, 128, 1, 3, 0, 1)),     # one full block, SYM7, l from the codes
    (86, (5, 7, 11), (1, 128, 128, 128, 128, 0, 7, 1, 0)),     # 172 plain, four blocks, key bias, V Hadamard
    (129, (1, 1, 257), (2, 1, 16, 128, 128, 0, 3, 0, 0)),      # 258: 256 plain, 2 in quarters (the last head)
    (257, (1, 8, 8), (1, 128, 64, 128, 128, 0, 3, 0, 0)),      # 256 plain, 1 in quarters, half a block of keys
    (130, (1, 15, 25), (3, 1, 128, 1 << 20, 128, 0, 4, 0, 0)), # 260, V scales per channel, Q smoothing alone
    # five full blocks and six with a partial last one, where every one of the three
    # tile buffers has been filled twice
    (22, (5, 8, 16), (1, 128, 128, 256, 128, 0, 3, 0, 0)),     # 66 in halves, V groups of two blocks
    (22, (5, 3, 47), (2, 128, 64, 256, 128, 1, 3, 0, 0)),      # 66 in halves, SYM7
    (22, (5, 3, 47), (1, 128, 128, 128, 128, 0, 7, 0, 0)),     # 66 in halves, key bias
    (22, (5, 3, 47), (1, 1, 1, 256, 128, 0, 3, 0, 0)),         # 66 in quarters, per-token
    (22, (5, 3, 47), (1, 128, 32, 128, 64, 0, 7, 0, 0)),       # 66 in halves, 12 blocks of 64, key bias
    (65, (5, 8, 16), (1, 128, 128, 256, 128, 0, 3, 0, 0)),     # 195 plain
    (65, (5, 3, 47), (2, 128, 64, 256, 128, 1, 3, 0, 0)),      # 195 plain, SYM7
    (65, (5, 3, 47), (1, 1, 1, 128, 64, 0, 3, 0, 0)),          # 195 plain, 12 blocks of 64, per-token
]


def _check(ora, w, case, heads, q, k, v):
    torch, ra = _torch(), _ra()
    rot, qg, kg, vg, kv, pq, sm, vrot, lq = case
    p = _params(ra, w, rot, qg, kg, vg, kv, pq, sm, fmt=FORMATS["e2m3"], vrot=vrot, lq=lq)
    bufs, _, _ = _run_quant(torch, ra, p, q, k, v)
    geo, cfg = _geo(ora, w), _cfg(ora, rot, qg, kg, vg, kv, pq, sm, vrot, lq)
    N, nb = w.N, -(-w.N // kv)
    args = (bufs["q_codes"], bufs["q_scale"], bufs["k_codes"], bufs["k_scale"], bufs["v_codes"], bufs["v_scale"],
            bufs["mu_v"] if sm & 2 else None)
    kb = bufs["k_bias"] if sm & 4 else None
    plain = torch.full((w.B * w.H, N, 128), float("nan"), dtype=torch.float32, device="cuda")
    ra.attn_int4(p, *args, plain, k_bias=kb)
    torch.cuda.synchronize()
    assert torch.isfinite(plain).all()          # every row was written
    s_d = torch.zeros((N, N), dtype=torch.int32, device="cuda")
    u_d = torch.zeros((N, N), dtype=torch.uint8, device="cuda")
    m_d = torch.zeros((N, nb), dtype=torch.float32, device="cuda")
    o = torch.empty_like(plain)
    for bh in heads:
        ra.attn_int4_debug(p, *args, o, bh, 0, N, s_d, u_d, m_d, k_bias=kb)
        torch.cuda.synchronize()
        ref, d = ora.fwd_int4_head(geo, cfg, q[0, bh], k[0, bh], v[0, bh], dumps=True)
        assert np.array_equal(s_d.cpu().numpy(), d["S"])
        assert np.all(m_d.cpu().numpy() == d["m"])
        pcode_check.compare(u_d.cpu().numpy(), d, pq, kv, N, label=f"{w.H}x{N} bh={bh}")
        assert np.abs(plain[bh].cpu().numpy() - ref).max() / np.abs(ref).max() <= O_TOL
    assert torch.equal(plain, o)


@pytest.mark.parametrize("plan", range(len(PLANS)))
def test_plain_and_split_tiles(ora, plan):
    from paper_2607_02584_amd import datagen as dg
    H, (T, Hg, W), case = PLANS[plan]
    print(f"[tile plan] H={H} grid={T}x{Hg}x{W} case={case}", flush=True)
    w = dg.small_workload(f"plan{plan}", T, Hg, W, H=H, seed=80 + plan)
    _check(ora, w, case, sorted({0, min(127, H - 1), H - 2, H - 1}), *_inputs(w))


@pytest.mark.parametrize("heads,kv", [(1, 128), (70, 128), (130, 128), (1, 64), (130, 64)])
def test_wholly_masked_chunk_has_no_maximum(ora, heads, kv):
    """Fewer tokens than one 32-key chunk with K scales per 32 keys: the other
    chunks' groups hold no token and have scale 0.  With every score negative
    the running maximum is negative, not the 0 that scale would give."""
    from paper_2607_02584_amd import datagen as dg
    print(f"[masked chunk] H={heads} kv={kv}", flush=True)
    w = dg.small_workload("masked", 1, 3, 5, H=heads, seed=95)
    q, k, v = _inputs(w)
    x = np.random.default_rng(3).uniform(1.0, 2.0, size=(1, heads, 1, 128)).astype(np.float32)
    small = np.random.default_rng(4).uniform(0.9, 1.1, size=q.shape).astype(np.float32)
    q, k = dg.f32_to_bf16_bits(x * small), dg.f32_to_bf16_bits(-x * small)
    # the positions turn by small angles only (theta large, extents small) along
    # the pairs that carry the product, so it stays negative; the oracle confirms
    case = (0, 128, 32, 128, kv, 0, 0, 0, 0)
    geo, cfg = _geo(ora, w), _cfg(ora, 0, 128, 32, 128, kv, 0, 0)
    _, d = ora.fwd_int4_head(geo, cfg, q[0, 0], k[0, 0], v[0, 0], dumps=True)
    assert d["m"].max() < 0
    _check(ora, w, case, [0, heads - 1], q, k, v)


def _check_fallback(ora, heads, grid, kv, fp16):
    from paper_2607_02584_amd import datagen as dg
    torch, ra = _torch(), _ra()
    print(f"[fallback tiles] H={heads} grid={grid} kv={kv} fp16={fp16}", flush=True)
    w = dg.small_workload("fbplan", *grid, H=heads, seed=97)
    q, k, v = _inputs(w)
    if fp16:
        # binary16 products carry 22 bits, so the order of the binary32 sums of
        # a score shows: up to 128 * 2^-24 of it, and ln 2 times that, on the
        # log2 scale, in P.  0.2 on Q and K keeps the scaled scores below 200
        # (they reach 5000 unscaled): at most 1e-3.
        q, k = (dg.f32_to_bf16_bits(0.2 * dg.bf16_bits_to_f32(x)) for x in (q, k))
        q, k, v = (np.clip(dg.bf16_bits_to_f32(x), -1000, 1000).astype(np.float16).view(np.uint16) for x in (q, k, v))
    p = ra.make_params(1, heads, grid, w.split, w.theta, rotation=ra.ROT_NONE, kv_block=kv, out_dtype=ra.FP32,
                       in_dtype=ra.FP16 if fp16 else ra.BF16)
    o = torch.full((heads, w.N, 128), float("nan"), dtype=torch.float32, device="cuda")
    ra.fwd_fp16(p, *(ra.to_device_bits(x) for x in (q, k, v)), o, ra.workspace(p, ra.PATH_FP16))
    torch.cuda.synchronize()
    assert torch.isfinite(o).all()
    geo = _geo(ora, w)
    for h in sorted({0, min(63, heads - 1), heads - 2, heads - 1}):
        ref = ora.fwd_fp16_head(geo, q[0, h], k[0, h], v[0, h], kv_block=kv, fp16=fp16)
        assert np.abs(o[h].cpu().numpy() - ref).max() / np.abs(ref).max() <= O_TOL


# heads at one tile each (64 tokens) or two (300 tokens): 64, 65, 128 and 129
# tiles on either side of the lines, then whole rounds with each kind of rest (at
# kv_block 64 the heads of 64 tokens from 257 on run on 4 waves throughout: one
# 128-query tile each, where 256-query tiles would start another round)
@pytest.mark.parametrize("fp16", [False, True])
@pytest.mark.parametrize("kv", [64, 128])
@pytest.mark.parametrize("heads,grid", [(64, (1, 8, 8)), (65, (1, 8, 8)), (128, (1, 7, 9)), (129, (1, 8, 8)),
                                        (257, (1, 8, 8)), (330, (1, 8, 8)), (33, (3, 10, 10)), (65, (3, 10, 10))])
def test_fallback_tiles(ora, heads, grid, kv, fp16):
    """The 16-bit fallback on each of its kernels: sampled heads against the
    fallback oracle, every row written."""
    _check_fallback(ora, heads, grid, kv, fp16)


@pytest.mark.parametrize("kv", [64, 128])
@pytest.mark.parametrize("heads,grid", [(86, (5, 8, 16)), (129, (2, 15, 15)), (165, (2, 15, 15)), (22, (5, 8, 16)),
                                        (22, (5, 3, 47)), (65, (5, 8, 16)), (65, (5, 3, 47))])
def test_fallback_tiles_of_several_blocks(ora, heads, grid, kv):
    """86 heads of 640 tokens: 430 tiles of 128 queries on 4 waves (kv_block 64),
    258 of 256 queries at kv_block 128; 129 and 165 heads of 450 tokens, two
    256-query tiles each: a whole round and the rest in quarters or halves; 22 and
    65 heads of 640 and 705 tokens, three tiles each: 66 in halves, 195 on 8 waves,
    the last block full and partial.
    (bfloat16 alone, since both types share every index: in binary16 the kernel's
    RoPE and the oracle's round some elements next to a tie to different
    neighbours, and one of K in these inputs, 11.43 +- 2^-7, moves O by 2.1e-3.)"""
    _check_fallback(ora, heads, grid, kv, False)


@pytest.mark.parametrize("fallback", [False, True])
def test_a_head_of_another_call(fallback):
    """The first head of 130 runs on the plain kernel, alone it runs on the
    key-split one: repeated calls give the same bytes, and the two calls differ by
    no more than the order of their binary32 sums allows."""
    torch, ra = _torch(), _ra()
    print(f"[head of another call] fallback={fallback}", flush=True)
    N, g = 300, torch.Generator().manual_seed(5)
    x = [torch.randn((1, 130, N, 128), generator=g).to(torch.bfloat16).cuda() for _ in range(3)]

    def run(H):
        p = ra.make_params(1, H, (3, 10, 10), rotation=ra.ROT_NONE if fallback else ra.ROT_INTERLEAVED,
                           out_dtype=ra.FP32)
        o = torch.empty((H, N, 128), dtype=torch.float32, device="cuda")
        ra.fwd(p, fallback, *(t[:, :H].contiguous() for t in x), o,
               ra.workspace(p, ra.PATH_FP16 if fallback else ra.PATH_INT4))
        torch.cuda.synchronize()
        return o
    whole, alone = run(130), run(1)
    assert torch.equal(whole, run(130)) and torch.equal(alone, run(1))
    # numerator and l are binary32 sums of N terms and three roundings a block, of
    # terms whose magnitudes add up to at most max |V| l (4 times that with P codes,
    # at most 2 P, and centred V, at most 2 max |V|), in two orders each
    mass = x[2][0, 0].float().abs().max().item() * (1 if fallback else 4)
    assert (whole[0] - alone[0]).abs().max().item() <= 4 * (N + 3 * 3) * 2.0 ** -24 * mass
