"""Every forward route on shapes chosen at the launch rules' boundaries, against
the oracle on sampled rows (codes, block exponents, row reference and
denominator through the test entry point; O and LSE through the forward).

The shapes reach every workgroup shape of every route: 256-query workgroups (wide),
128-query workgroups of four waves (narrow), and eight waves that split the keys of 128
(half), 64 (quarter) or 32 (eighth) queries.  The comments name the shape of the plain
route (which the guarded and exponential routes share) and, where it differs, of the
causal, FP8 P/V and causal FP8 routes; a CPU test of the launch rules holds the two tables
to every kernel that the rules can launch, over enough keys that its main loop runs.
Rows: the first and last of the tensor and of a head, and seeded random ones.  Also the
largest shapes of the paper's D128 and D64 tables, which the benchmark times."""
import numpy as np
import pytest
import torch

import workloads
from test_gpu_forward import _run_and_check, _run_fp8, _run_guarded

pytestmark = pytest.mark.gpu

SHAPES = [  # B, H, N, d
    (1, 32, 2048, 128),    # wide: one full round of 256; causal narrow, causal FP8 half
    (1, 257, 256, 128),    # narrow: 257 wide workgroups would start a second round; FP8 wide
    (5, 64, 256, 128),     # narrow: a second round of 64; FP8 wide
    (2, 40, 1536, 128),    # wide: a second round of 224; causal narrow
    (1, 1290, 256, 128),   # wide: six rounds; causal narrow
    (3, 7, 1664, 128),     # narrow: N = 13 x 128; FP8 half
    (2, 3, 4224, 64),      # half: N = 33 x 128; causal quarter
    (1, 3, 12288, 128),    # wide: 144 workgroups, fewer than the CUs; causal half
    (1, 6, 8320, 64),      # half: N = 65 x 128; FP8 narrow
    (1, 16, 4096, 64),     # half: at most two workgroups of 128 queries per CU; FP8 narrow
    (1, 768, 1024, 64),    # wide: 3072 of them, causal too; FP8 narrow
    (1, 1, 128, 128),      # narrow: one tile; FP8 half
    (1, 40, 2048, 64),     # narrow on every route
    (1, 22, 768, 128),     # narrow, FP8 too: fewer workgroups than CUs, rows too short to split; causal FP8 half
    (1, 24, 4096, 128),    # narrow; causal wide, FP8 half
]


def _inputs(B, H, N, d):
    g = torch.Generator().manual_seed(B * 1000003 + H * 1009 + N * 7 + d)
    q, k, v = (torch.randn(B, H, N, d, generator=g).to(torch.bfloat16) for _ in range(3))
    host64 = tuple(workloads.as_f64(t) for t in (q, k, v))
    rows = np.random.default_rng(N + H).integers(0, B * H * N, 40)
    rows = np.unique(np.concatenate([rows, [0, N - 1, B * H * N - N, B * H * N - 1]]))
    return host64, (q.cuda(), k.cuda(), v.cuda()), rows


@pytest.mark.parametrize("B,H,N,d", SHAPES)
def test_every_route_at_launch_boundaries(B, H, N, d):
    import paper_2609_04105_amd as fa
    host64, dev, rows = _inputs(B, H, N, d)
    label = f"sweep B{B} H{H} N{N} d{d}"
    _run_and_check(fa, host64, dev, rows, label)
    _run_and_check(fa, host64, dev, rows, label + " causal", causal=True, lse=True)
    _run_and_check(fa, host64, dev, rows, label + " ex2 4", ex2_pairs=4)
    _run_guarded(fa, host64, dev, rows, label + " guard", 110, 16)
    _run_fp8(fa, host64, dev, rows, label + " fp8")
    _run_fp8(fa, host64, dev, rows, label + " fp8 causal", causal=True)


# Launches that split the keys of a workgroup's queries among its waves: tile counts that
# leave key groups one stage short or without work, one to several turns of the ring.  (FP8
# P/V with d = 128 takes quarter in the place of eighth.)
SPLIT_SHAPES = [
    (1, 1, 512, 128),      # eighth, one stage of four tiles
    (1, 2, 640, 128),      # eighth, five tiles: one group of four has a tile in the second stage
    (1, 2, 640, 64),       # quarter, three stages of two tiles, the last half filled
    (1, 3, 1152, 64),      # eighth, nine tiles
    (1, 1, 4224, 128),     # eighth, 33 tiles (causal: 32-query workgroups ending in every tile)
    (1, 1, 4224, 64),      # the same, with a ring of four stages
    (3, 7, 640, 64),       # quarter, 105 workgroups of 128 queries
    (1, 16, 640, 128),     # quarter, three stages, the last half filled
    (1, 4, 3200, 128),     # quarter, 25 tiles
    (1, 4, 3200, 64),      # the same, one step deep
    (1, 9, 2176, 128),     # half, 17 tiles
    (2, 5, 1664, 64),      # half, 13 tiles
    (1, 12, 2048, 64),     # half, 192 workgroups
    (1, 5, 5120, 64),      # half; causal quarter over 200 workgroups
    (1, 3, 14080, 128),    # causal half over 330 workgroups; plain and FP8 wide
    (1, 20, 4096, 128),    # FP8 half, where wide would take a second round; plain narrow, causal FP8 wide
]


@pytest.mark.parametrize("B,H,N,d", SPLIT_SHAPES)
def test_every_route_with_split_keys(B, H, N, d):
    import paper_2609_04105_amd as fa
    host64, dev, rows = _inputs(B, H, N, d)
    label = f"split B{B} H{H} N{N} d{d}"
    _run_and_check(fa, host64, dev, rows, label, lse=True)
    _run_and_check(fa, host64, dev, rows, label + " causal", causal=True, lse=True)
    _run_and_check(fa, host64, dev, rows, label + " ex2 16", ex2_pairs=16)
    _run_guarded(fa, host64, dev, rows, label + " guard", 110, 16)
    _run_fp8(fa, host64, dev, rows, label + " fp8")
    _run_fp8(fa, host64, dev, rows, label + " fp8 causal", causal=True)


# Grids of the same heads that reach every workgroup shape: N, and the number of heads.
GRIDS = {64: (2048, (2, 8, 16, 40, 64, 384)), 128: (4096, (2, 4, 8, 10, 20, 24))}
OPTIONS = ([dict(ex2_pairs=x) for x in (0, 1, 2, 4, 8, 16)] + [dict(guard=(110, 16), ex2_pairs=x) for x in (0, 4, 16)]
           + [dict(causal=True, ex2_pairs=x) for x in (0, 4, 16)] + [dict(pv_fp8=True), dict(pv_fp8=True, causal=True)])


@pytest.mark.parametrize("d", GRIDS)
def test_every_option_is_the_same_on_every_grid(d):
    """Two heads, alone and repeated over grids that take the other workgroup shapes, with
    every option that has kernels of its own: codes do not depend on the shape, so only the
    order of the fp32 sums differs (at most 64 additions of 64-key products per output: a
    rounding walk of sqrt(64) 2^-24 = 5e-7, gate 1e-5)."""
    import paper_2609_04105_amd as fa
    N, grids = GRIDS[d]
    g = torch.Generator(device="cuda").manual_seed(d)
    q, k, v = (torch.randn((1, 2, N, d), device="cuda", generator=g) for _ in range(3))
    k[:, :, ::256] *= 6.0            # references that differ between key groups
    for opts in OPTIONS:
        ops = fa.quantize_qkv(q, k, v, anchored="guard" in opts, pv_fp8=opts.get("pv_fp8", False))
        want = want_lse = None
        for H in grids:
            print(f"[grids] d{d} N{N} H{H} {opts}", flush=True)
            lse = torch.full((1, H, N), float("nan"), device="cuda")
            out = fa.forward_mxfp4(*(t.repeat(1, H // 2, 1, 1) for t in ops), lse=lse, **opts)
            out, lse = out.view(H // 2, 2, N, d).double(), lse.view(H // 2, 2, N)
            if want is None:
                want, want_lse = out, lse
                assert bool(torch.isfinite(want).all())
            rel = ((out - want).flatten(1).norm(dim=1) / want.norm()).max().item()
            assert rel <= 1e-5, (opts, H, rel)
            assert (lse - want_lse).abs().max().item() <= 1e-5 * max(1.0, want_lse.abs().max().item()), (opts, H)


@pytest.mark.parametrize("H,N,d", [(24, 32768, 128), (64, 32768, 64)])
def test_paper_largest_shapes_sampled_rows(H, N, d):
    """The largest shapes of the paper's D128 and D64 tables (B1), in the launch the
    benchmark times (wide workgroups; at d = 64 two per CU, four waves per SIMD): bf16 N(0,1) inputs drawn on the GPU, 24 rows from six
    heads (the first and last of the sequence among them) against the oracle."""
    import paper_2609_04105_amd as fa
    g = torch.Generator(device="cuda").manual_seed(N + H + d)
    q, k, v = (torch.randn((1, H, N, d), device="cuda", generator=g).to(torch.bfloat16) for _ in range(3))
    rng = np.random.default_rng(H + d)
    heads = np.unique(np.concatenate([[0, H - 1], rng.integers(0, H, 4)]))
    rows = np.unique(np.concatenate([h * N + np.concatenate([[0, N - 1], rng.integers(0, N, 3)]) for h in heads]))
    sel = torch.from_numpy(np.unique(heads)).cuda()
    # the oracle sees only the heads the rows touch, renumbered 0..len(heads)-1
    host64 = tuple(workloads.as_f64(t[:, sel].cpu()) for t in (q, k, v))
    remap = {int(h): i for i, h in enumerate(np.unique(heads))}
    local = np.array([remap[int(r // N)] * N + int(r % N) for r in rows])
    print(f"[paper shape B1 H{H} N{N} d{d}] rows={len(rows)} heads={len(heads)}", flush=True)
    out = fa.forward_mxfp4(*fa.quantize_qkv(q, k, v))
    torch.cuda.synchronize()
    got = out.reshape(-1, d)[torch.from_numpy(rows).cuda()].cpu().numpy().astype(np.float64)
    from parity import check_output, oracle_rows
    ref = oracle_rows(*host64, local, 1.0 / np.sqrt(d), want_codes=False)
    check_output(got, ref["O"], f"paper shape B1 H{H} N{N} d{d}")
