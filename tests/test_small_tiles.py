"""Products in small tiles (lists that leave the chip idle at the usual ones).

CPU: the planner's choice and its tile lists (``planner_small_tiles_driver.cpp``).
GPU: Muon steps over the same lists against the oracle, at sides on both
sides of a tile edge and K loops of one stage, of fewer stages than a tile has
LDS buffers. A bf16 matrix has the same result, to the bit, in every list.
"""
import os
import shutil
import subprocess

import numpy as np
import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_2605_19811_amd", "csrc")

# list of shapes -> "tile/LDS stages" of Gram, polynomial, apply
# (0: the usual tiles)
LISTS = {
    "one-stage": ([(64, 64)], "64/8 64/8 64/2"),
    "edges": ([(65, 129), (129, 65), (127, 193), (64, 321)], "64/8 64/8 64/2"),
    "one-wide": ([(300, 1000)], "64/8 64/8 64/2"),
    "one-tall": ([(1089, 257)], "64/8 64/8 64/2"),
    "two-per-cu": ([(500, 700), (700, 500)] * 5, "64/4 64/4 64/2"),
    "apply-128": ([(768, 2304), (768, 768), (768, 3072), (3070, 766)], "64/4 64/4 128/2"),
    "poly-two-stage": ([(2000, 2000)], "64/2 64/2 64/2"),
    "gram-small-only": ([(768, 2304), (768, 768), (768, 3072), (3072, 768)] * 3, "64/4 0/2 0/2"),
    # small tiles for one product and the usual ones for the next, which then read
    # padding that the small ones did not write
    "ragged-gram-only": ([(765, 2300), (765, 765), (765, 3070), (3070, 765)] * 3, "64/4 0/2 0/2"),
    "ragged-apply-usual": ([(901, 2703), (901, 901), (901, 3604), (3604, 901)], "64/4 64/4 0/2"),
}


@pytest.fixture(scope="module")
def planner(tmp_path_factory):
    if shutil.which("g++") is None:
        pytest.skip("needs g++")
    exe = str(tmp_path_factory.mktemp("planner") / "small_tiles")
    subprocess.run(["g++", "-O1", "-std=c++17", f"-I{CSRC}",
                    os.path.join(HERE, "planner_small_tiles_driver.cpp"),
                    os.path.join(CSRC, "plan.cpp"), "-o", exe], check=True)

    def run(shapes, prec="bf16"):
        args = [str(v) for s in shapes for v in s]
        out = subprocess.run([exe, prec, *args], capture_output=True, text=True)
        assert out.returncode == 0, out.stdout
        return out.stdout
    return run


def test_planner_small_tile_lists(planner):
    for name, (shapes, variants) in LISTS.items():
        assert planner(shapes).split("bad")[0].strip() == variants, name
    # (the list of test_noalloc_where_only_the_usual_tiles_fit)
    assert planner([(1792, 7424), (256, 512)]).startswith("64/4 64/4 0/2")
    for name, (shapes, variants) in F32_LISTS.items():
        assert planner(shapes, "fp32").split("bad")[0].strip() == variants, name


# A plan is built anew wherever list signatures alternate beyond those that are
# kept: choosing the tiles stays a small part of it on large sets, and of the order
# of the rest on short lists (1.0 and 2-3 measured; 5-20 when every variant's lists
# were built to be estimated).
@pytest.mark.parametrize("layers,most", [(1, 6.0), (12, 2.0), (24, 2.0)])
def test_choosing_small_tiles_is_cheap(planner, layers, most):
    shapes = [(768, 2304), (768, 768), (768, 3072), (3072, 768)] * layers
    assert float(planner(shapes).split("cost")[1]) < most


@pytest.mark.gpu
@pytest.mark.parametrize("name", sorted(LISTS))
def test_small_tiles_match_oracle(name):
    import torch

    from paper_2605_19811_amd import lionmuon as lm
    from parity import check_muon
    shapes = LISTS[name][0]
    rng = np.random.default_rng(len(shapes) + shapes[0][0])
    W0, M0, G = ([(rng.standard_normal(s) * std).astype(np.float32) for s in shapes]
                 for std in (0.02, 1e-2, 1e-2))
    W, M, Gd = ([torch.from_numpy(x).cuda() for x in t] for t in (W0, M0, G))
    cfg = lm.config(lr_muon=0.02)
    # a workspace of NaN: what no kernel of the call writes must not be read
    ws = torch.full((lm.lionmuon_workspace_bytes([(*s, False) for s in shapes], cfg),), 0xFF,
                    dtype=torch.uint8, device="cuda")
    lm.lionmuon_step_ex(W, Gd, M, 0, 1, 0.9, 0.99, 0.1, cfg, workspace=ws)
    torch.cuda.synchronize()
    for i in range(len(shapes)):
        check_muon(W0[i], G[i], M0[i], W[i].cpu().double().numpy(), M[i].cpu().double().numpy(),
                   0.9, 0.99, 0.02, 0.1, "bf16")


# A bf16 matrix alone and 40 or more of it in one call, which run in other tiles
# (K loops of 1 to 48 stages, below and above the eight LDS stages of a tile
# alone on its CU; edges of 64-tiles): each element's sum runs through K in
# order in either, so the results are equal.
SAME = {(64, 64): 512, (65, 448): 256, (96, 512): 256, (128, 577): 256, (256, 1024): 256,
        (300, 1000): 192, (1000, 300): 192, (768, 3072): 40}


@pytest.mark.gpu
@pytest.mark.parametrize("shape", sorted(SAME))
def test_bf16_result_does_not_depend_on_the_list(shape):
    import torch

    from paper_2605_19811_amd import lionmuon as lm
    gen = torch.Generator(device="cuda")
    gen.manual_seed(shape[0])
    x = torch.randn((SAME[shape], *shape), generator=gen, device="cuda")
    cfg = lm.config()
    many = lm.lionmuon_ns(x, cfg)
    for i in (0, SAME[shape] - 1):
        assert torch.equal(lm.lionmuon_ns(x[i].contiguous(), cfg), many[i])


# fp32 products: K loops of 1 to 9 and 18 stages of 64 on 64-tiles (a round is 8),
# tile edges, the apply alone on 128-tiles, and all three products on 128-tiles
# with 47 and 63 stages of 32 (odd, and no multiple of a round's four)
F32_LISTS = {
    "one-stage": ([(2, 3), (33, 64), (64, 40)], "64/2 64/2 64/2"),
    "edges": ([(65, 129), (129, 193), (257, 191), (63, 449)], "64/2 64/2 64/2"),
    "rounds": ([(512, 513), (577, 513), (100, 1089)], "64/2 64/2 64/2"),
    "apply-128": ([(1000, 3000), (1000, 3000)], "64/2 64/2 128/2"),
    "tile-128": ([(1500, 2000), (2000, 1500)], "128/2 128/2 128/2"),
}


@pytest.mark.gpu
@pytest.mark.parametrize("name", sorted(F32_LISTS))
def test_split_fp32_products_match_oracle(name):
    import torch

    from paper_2605_19811_amd import lionmuon as lm
    from parity import check_muon
    shapes = F32_LISTS[name][0]
    rng = np.random.default_rng(len(shapes) + shapes[0][0])
    W0, M0, G = ([(rng.standard_normal(s) * std).astype(np.float32) for s in shapes]
                 for std in (0.02, 1e-2, 1e-2))
    W, M, Gd = ([torch.from_numpy(x).cuda() for x in t] for t in (W0, M0, G))
    cfg = lm.config(ns_precision="fp32", lr_muon=0.02)
    ws = torch.full((lm.lionmuon_workspace_bytes([(*s, False) for s in shapes], cfg),), 0xFF,
                    dtype=torch.uint8, device="cuda")
    lm.lionmuon_step_ex(W, Gd, M, 0, 1, 0.9, 0.99, 0.1, cfg, workspace=ws)
    torch.cuda.synchronize()
    for i in range(len(shapes)):
        check_muon(W0[i], G[i], M0[i], W[i].cpu().double().numpy(), M[i].cpu().double().numpy(),
                   0.9, 0.99, 0.02, 0.1, "fp32")


def newton_schulz_batch(x, dtype):
    """Five quintic steps of a batch of wide matrices in plain numpy."""
    a, b, c = (dtype(v) for v in (3.4445, -4.7750, 2.0315))
    norm = np.sqrt(np.square(x.astype(np.float64)).sum((1, 2), keepdims=True)) + 1e-7
    x = x.astype(dtype) / norm.astype(dtype)
    for _ in range(5):
        g = x @ x.transpose(0, 2, 1)
        x = (a * np.eye(x.shape[1], dtype=dtype) + (b * g + c * (g @ g))) @ x
    return x.astype(np.float64)


@pytest.mark.gpu
@pytest.mark.parametrize("count", [1500, 2500])          # 64-tiles, 128-tiles
@pytest.mark.parametrize("shape", [(2, 3), (2, 64), (3, 17), (4, 8), (8, 16), (16, 150), (48, 96)])
def test_fp32_products_are_as_exact_as_32_bit_sums(shape, count):
    """Short sides, where dropped parts of a product show most: over many
    matrices, no further from 64 bits than the recursion in 32-bit numpy is."""
    import torch

    from paper_2605_19811_amd import lionmuon as lm
    count //= max(1, shape[0] * shape[1] // 1000)        # (the large ones: fewer do)
    x = np.random.default_rng(shape[0]).standard_normal((count, *shape)).astype(np.float32)
    o = lm.lionmuon_ns(torch.from_numpy(x).cuda(), lm.config(ns_precision="fp32")).cpu().double().numpy()
    ref = newton_schulz_batch(x, np.float64)
    assert np.linalg.norm(o - ref) <= np.linalg.norm(newton_schulz_batch(x, np.float32) - ref)


@pytest.mark.gpu
@pytest.mark.parametrize("prec,tol", [("bf16", 2e-2), ("fp32", 1e-4)])
@pytest.mark.parametrize("shape", [(65, 131), (131, 65), (200, 333), (333, 200)])
def test_rows_off_16_bytes(shape, prec, tol):
    """Rows that no 16-byte access divides: the hook's store and a step on
    buffers one float off (tolerances: the two precisions' error budgets)."""
    import torch

    import oracle
    from paper_2605_19811_amd import lionmuon as lm
    from parity import check_muon
    rng = np.random.default_rng(shape[0])
    W0, M0, G = ((rng.standard_normal(shape) * std).astype(np.float32) for std in (0.02, 1e-2, 1e-2))
    cfg = lm.config(ns_precision=prec, lr_muon=0.02)
    o = lm.lionmuon_ns(torch.from_numpy(G).cuda(), cfg).cpu().double().numpy()
    ref = oracle.newton_schulz(G)
    assert np.linalg.norm(o - ref) <= tol * np.linalg.norm(ref)

    def off(x):
        flat = torch.full((x.size + 2,), float("nan"), device="cuda")
        flat[1:-1] = torch.from_numpy(x.ravel()).cuda()
        return flat, flat[1:-1].view(*shape)
    (fw, W), (_, Gd), (fm, M) = off(W0), off(G), off(M0)
    lm.lionmuon_step_ex([W], [Gd], [M], 0, 1, 0.9, 0.99, 0.1, cfg)
    torch.cuda.synchronize()
    for flat in (fw, fm):                       # nothing written past either end
        assert torch.isnan(flat[0]) and torch.isnan(flat[-1])
    check_muon(W0, G, M0, W.cpu().double().numpy(), M.cpu().double().numpy(),
               0.9, 0.99, 0.02, 0.1, prec)


@pytest.mark.gpu
@pytest.mark.parametrize("prec", ["bf16", "fp32"])
@pytest.mark.parametrize("shape", [(65, 132), (64, 600), (300, 1000), (132, 68), (600, 200), (1000, 300)])
def test_result_does_not_depend_on_where_a_matrix_starts(shape, prec):
    """The same step on 16-byte aligned buffers and on buffers one float off:
    every sum has one order, so W and M are equal to the bit."""
    import torch

    from paper_2605_19811_amd import lionmuon as lm
    gen = torch.Generator(device="cuda")
    gen.manual_seed(shape[0])
    x = [torch.randn(shape, generator=gen, device="cuda") * std for std in (0.02, 1e-2, 1e-2)]
    cfg = lm.config(ns_precision=prec, lr_muon=0.02)
    out = []
    for shift in (0, 1):
        W, G, M = (torch.empty(v.numel() + 4, device="cuda")[shift:shift + v.numel()].view(shape).copy_(v)
                   for v in x)
        lm.lionmuon_step_ex([W], [G], [M], 0, 1, 0.9, 0.99, 0.1, cfg)
        out.append((W, M))
    assert torch.equal(out[0][1], out[1][1]) and torch.equal(out[0][0], out[1][0])
