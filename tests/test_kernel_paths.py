"""Every wave-K tile, every K-tail form and the guarded kernel, each on products that the library itself sends there.

Which sizes run on which kernel is up to the time models and may change with them; so the products are searched for
here (host logic only) by the names of the kernels that would run, and a kernel that no product reaches fails."""
import math
import random
import re
import shutil
import subprocess
from functools import lru_cache

import numpy as np
import pytest
import torch

from paper_2502_08145_amd import binding as B
from paper_2502_08145_amd import synth
from paper_2502_08145_amd.profile_summary import kernel_key, short

LAYOUTS = ["NN", "NT", "TN"]


def _log_int(rng, lo, hi, step):
    return max(step, round(math.exp(rng.uniform(math.log(lo), math.log(hi))) / step) * step)


@lru_cache(maxsize=None)
def reached():
    """{(kernel name with its wave count, layout): [the two smallest sampled products of one launch on it]}"""
    rng = random.Random(20250208)
    found = {}
    for _ in range(30000):
        step = rng.choice([1, 8, 8, 8])
        M, N, K = (_log_int(rng, lo, 4200, step) for lo in (16, 16, 24))
        if not 2e6 < M * N * K < 1e10:
            continue
        for layout in LAYOUTS:
            names = B.kernels(M, N, K, layout)
            if len(names) == 1 and (names[0].startswith(("wavek", "edge")) or names[0].endswith("_ktail")):
                best = found.setdefault((names[0], layout), [])
                best.append((M, N, K))
                best.sort(key=lambda s: s[0] * s[1] * s[2])
                del best[2:]
    return found


def test_every_such_kernel_of_the_library_is_reached():
    nm = shutil.which("nm")
    if not nm:
        pytest.skip("nm is missing")
    out = subprocess.run([nm, "-C", B.LIB_PATH], capture_output=True, text=True, check=True).stdout
    built = {short(m.group(1)) for m in re.finditer(r"axonn::__device_stub__(.*)", out)}
    built = {n for n in built if n.startswith(("wavek", "edge")) or "_ktail" in n}
    have = {kernel_key(name, layout) for name, layout in reached()}
    assert built == have, (built - have, have - built)


def _bits(bits):
    return torch.from_numpy(np.ascontiguousarray(bits).view(np.int16)).cuda().view(torch.bfloat16)


def _check(oracle_mod, M, N, K, layout, kernels):
    """Integers of |value| <= 4 are exact in fp32 in any order (|sum| <= 16 K < 2^24): every element, and nothing
    behind the output.  The device's fp32 product that they are compared with is checked against the oracle."""
    a, b = synth.integer_bf16(910 + M, (M, K), -4, 4), synth.integer_bf16(920 + N, (K, N), -4, 4)
    A = synth.transpose_bits(a) if layout == "TN" else a
    Bm = synth.transpose_bits(b) if layout == "NT" else b
    ref = _bits(a).float() @ _bits(b).float()
    rng = np.random.default_rng(M + N + K)
    ii, jj = rng.integers(0, M, 64), rng.integers(0, N, 64)
    ii[:4], jj[:4] = (0, 0, M - 1, M - 1), (0, N - 1, 0, N - 1)
    at = oracle_mod.gemm_at(M, N, K, layout, A, Bm, ii, jj)
    assert np.array_equal(ref[torch.from_numpy(ii).cuda(), torch.from_numpy(jj).cuda()].cpu().numpy(), at)
    assert B.kernels(M, N, K, layout, now=True) == kernels
    c = torch.empty((M + 2, N), dtype=torch.bfloat16, device="cuda")
    c.view(torch.int16).fill_(0x7FC0)
    x, y = _bits(A), _bits(Bm)
    B.axonn_linear_fwd(M, N, K, layout, x, y, c[:M])
    torch.cuda.synchronize()
    got = c[:M].clone()
    assert torch.equal(got.view(torch.int16), ref.to(torch.bfloat16).view(torch.int16)), (kernels, layout, (M, N, K))
    assert bool((c[M:].view(torch.int16) == 0x7FC0).all())
    for _ in range(2):   # the same bits again
        B.axonn_linear_fwd(M, N, K, layout, x, y, c[:M])
    torch.cuda.synchronize()
    assert torch.equal(got.view(torch.int16), c[:M].view(torch.int16))


@pytest.mark.gpu
@pytest.mark.parametrize("family", ["wavek_16x16", "wavek_16x32", "wavek_32x32", "wavek_32x64", "wavek_64x64", "ktail", "edge"])
@pytest.mark.parametrize("layout", LAYOUTS)
def test_kernels_on_products_that_reach_them(oracle_mod, layout, family):
    B.register_workspace()
    cases = [(name, s) for (name, lay), shapes in sorted(reached().items()) if lay == layout and family in name for s in shapes]
    for name, (M, N, K) in cases:
        print(f"  {name} {layout} {(M, N, K)}", flush=True)
        _check(oracle_mod, M, N, K, layout, [name])


@lru_cache(maxsize=None)
def small_tile_products(kernel, layout):
    """Products of one launch on `kernel`: up to one each of the shortest K (all of it in LDS), of one to six steps more (either
    parity, the ring once around) and of some dozens, on outputs of whole and of ragged tiles.  (The 128 x 128 tile in two
    groups is taken for a long K only.)"""
    rng = random.Random(f"{kernel} {layout}")
    found = {}
    long_k = "128x128" in kernel
    for _ in range(40000):
        steps = rng.choice([32, 33, 47, 48, 65] if long_k else [2, 3, 4, 5, 6, 7, 8, 9, 24, 25, 33])
        step = rng.choice([8, 64])
        M, N, K = _log_int(rng, 1024 if long_k else 64, 2304, step), _log_int(rng, 1024 if long_k else 64, 2304, step), 64 * steps
        if B.kernels(M, N, K, layout) == [kernel]:
            key = (steps, M % 64 == 0 and N % 64 == 0)
            if key not in found or M * N < found[key][0] * found[key][1]:
                found[key] = (M, N, K)
    return sorted(found.values())


@pytest.mark.gpu
@pytest.mark.parametrize("layout", LAYOUTS)
@pytest.mark.parametrize("kernel", ["mfma16k64g_64x64_g2", "mfma16k64g_64x128", "mfma16k64g_128x64", "mfma16k64g_128x128_g2"])
def test_small_tiles_of_the_eight_wave_kernel(oracle_mod, layout, kernel):
    if kernel == "mfma16k64g_128x128_g2" and layout == "NT":
        pytest.skip("not built: one group is as fast there")
    B.register_workspace()
    shapes = small_tile_products(kernel, layout)
    assert shapes
    for shape in shapes:
        print(f"  {kernel} {layout} {shape}", flush=True)
        _check(oracle_mod, *shape, layout, [kernel])


@lru_cache(maxsize=None)
def eight_wave_products():
    """{(kernel, layout): {64-k steps: the smallest sampled product of one launch on it}}, K a multiple of 64 or, for the "_ktail" forms,
    not (any K for TN, multiples of 8 where an operand is K-contiguous)."""
    rng = random.Random(16)
    found = {}
    for _ in range(60000):
        layout, steps, step = rng.choice(LAYOUTS), rng.choice([2, 3, 4, 5, 6, 7, 8, 9, 24, 25, 33, 48, 65]), rng.choice([8, 8, 64])
        M, N, K = _log_int(rng, 64, 6000, step), _log_int(rng, 64, 6000, step), 64 * steps
        if rng.random() < 0.6:
            K -= rng.randrange(1, 64) if layout == "TN" and rng.random() < 0.5 else 8 * rng.randrange(1, 8)
        if M * N * K > 2e10:
            continue
        names = B.kernels(M, N, K, layout)
        if len(names) == 1 and names[0].startswith("mfma16k64g"):
            best = found.setdefault((names[0], layout), {})
            if steps not in best or M * N < best[steps][0] * best[steps][1]:
                best[steps] = (M, N, K)
    return found


@pytest.mark.gpu
@pytest.mark.parametrize("layout", LAYOUTS)
@pytest.mark.parametrize("tail", ["", "_ktail"])
@pytest.mark.parametrize("tile", ["64x64_g2", "64x128", "128x64", "128x128", "256x128", "128x256"])
def test_every_length_of_k_on_the_eight_wave_kernel(oracle_mod, tile, tail, layout):
    """The ring has three to five stages: a K that is shorter, exactly as long, and up to three steps longer (refills, window and
    waits, either parity), and some dozens of steps, with a shorter last 64 k, which is staged first, and without."""
    kernel = f"mfma16k64g_{tile}{tail}"
    products = eight_wave_products()[(kernel, layout)]
    assert len(set(products) & {2, 3, 4, 5, 6, 7, 8, 9}) >= 7 and max(products) >= 24, products
    B.register_workspace()
    for steps, shape in sorted(products.items()):
        print(f"  {kernel} {layout} {shape}", flush=True)
        _check(oracle_mod, *shape, layout, [kernel])


@pytest.mark.gpu
@pytest.mark.parametrize("layout", LAYOUTS)
@pytest.mark.parametrize("tail", ["", "_ktail"])
@pytest.mark.parametrize("tile", ["96x128", "192x128"])
def test_tiles_of_96_and_192_rows(oracle_mod, tile, tail, layout):
    """Loads for a part of a wave (12 rows a wave of a K-contiguous operand; k-rows that LDS holds padded): every length of K there is a product of."""
    kernel = f"mfma16k64g_{tile}{tail}"
    products = eight_wave_products()[(kernel, layout)]
    assert len(set(products) & {2, 3, 4, 5, 6, 7, 8, 9}) >= 4 and max(products) >= 24, products
    B.register_workspace()
    for steps, shape in sorted(products.items()):
        print(f"  {kernel} {layout} {shape}", flush=True)
        _check(oracle_mod, *shape, layout, [kernel])


@lru_cache(maxsize=None)
def by_lines_products():
    """{(kernel, layout): {pieces of 8 beyond whole 64 k: the smallest sampled product of one launch on it}}, K beyond 768."""
    rng = random.Random(17)
    found = {}
    for _ in range(60000):
        layout, K = rng.choice(["NN", "NT"]), 8 * rng.randrange(97, 300)
        M, N = _log_int(rng, 64, 4000, 8), _log_int(rng, 64, 4000, 8)
        names = B.kernels(M, N, K, layout)
        if K % 64 and len(names) == 1 and names[0].startswith("mfma16k64g"):
            best, left = found.setdefault((names[0], layout), {}), K % 64 // 8
            if left not in best or M * N * K < math.prod(best[left]):
                best[left] = (M, N, K)
    return found


@pytest.mark.gpu
@pytest.mark.parametrize("layout", ["NN", "NT"])
@pytest.mark.parametrize("tile", ["64x64_g2", "64x128", "128x64", "96x128", "128x128"])
def test_k_contiguous_rows_loaded_by_lines(tile, layout):
    """Rows that start on every 16 bytes of a line (each K modulo 64, buffers on every 16 bytes of one): integers, exact in any order."""
    B.register_workspace()
    products = by_lines_products()[(f"mfma16k64g_{tile}_ktail", layout)]
    assert set(products) == set(range(1, 8)), products
    for left, (M, N, K) in products.items():
        for at_a, at_b in ((left, 0), (3, left), (0, 8 - left)):
            print(f"  {tile} {layout} {(M, N, K)} {at_a} {at_b}", flush=True)
            a = torch.randint(-4, 5, (8 * at_a + M * K,), device="cuda").to(torch.bfloat16)[8 * at_a:].view(M, K)
            b = torch.randint(-4, 5, (8 * at_b + N * K,), device="cuda").to(torch.bfloat16)[8 * at_b:].view(*((N, K) if layout == "NT" else (K, N)))
            c = torch.full((M + 2, N), float("nan"), dtype=torch.bfloat16, device="cuda")
            B.axonn_linear_fwd(M, N, K, layout, a, b, c[:M])
            ref = a.float() @ (b.float().t().contiguous() if layout == "NT" else b.float())
            assert torch.equal(c[:M], ref.to(torch.bfloat16)) and bool(c[M:].isnan().all())


@lru_cache(maxsize=None)
def eight_wave_split_products():
    """{(kernel, layout): the smallest sampled product of one launch on it} with the whole scratch area registered; ranges of equal length
    and not, from a few 64 k to some dozens."""
    rng = random.Random(18)
    found = {}
    for _ in range(30000):
        layout, M, N, K = rng.choice(LAYOUTS), *(_log_int(rng, 128, 4096, 128) for _ in range(2)), _log_int(rng, 512, 24000, 64)
        if M * N > 1 << 22 or M * N * K > 3e10:
            continue
        names = B.kernels(M, N, K, layout, now=True)
        if len(names) == 1 and re.match(r"mfma16k64g_\d+x\d+_sk", names[0]):
            best = found.setdefault((names[0], layout), (M, N, K))
            if M * N * K < math.prod(best):
                found[(names[0], layout)] = (M, N, K)
    return found


@pytest.mark.gpu
@pytest.mark.parametrize("layout", LAYOUTS)
def test_split_k_on_the_eight_wave_kernel(oracle_mod, layout):
    """Every tile and number of K ranges that the library picks: every element, the flags taken back, the same bits again, and from a
    captured graph, which carries one epoch through its replays."""
    area = B.register_workspace()
    products = {name: shape for (name, lay), shape in eight_wave_split_products().items() if lay == layout}
    assert {n.split("_sk")[0] for n in products} >= {"mfma16k64g_64x128", "mfma16k64g_128x128"}, products
    assert {int(n.split("_sk")[1]) for n in products} >= {2, 3, 4, 5}, products
    for name, (M, N, K) in sorted(products.items()):
        print(f"  {name} {layout} {(M, N, K)}", flush=True)
        _check(oracle_mod, M, N, K, layout, [name])
    name, (M, N, K) = min(products.items(), key=lambda p: math.prod(p[1]))
    x = torch.randn((K, M) if layout == "TN" else (M, K), device="cuda").to(torch.bfloat16)
    y = torch.randn((N, K) if layout == "NT" else (K, N), device="cuda").to(torch.bfloat16)
    want, c = (torch.empty((M, N), dtype=torch.bfloat16, device="cuda") for _ in range(2))
    B.axonn_linear_fwd(M, N, K, layout, x, y, want)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        for _ in range(2):
            B.axonn_linear_fwd(M, N, K, layout, x, y, c)
    for _ in range(4):
        c.zero_()
        graph.replay()
        B.axonn_linear_fwd(M, N, K, layout, x, y, want)
        torch.cuda.synchronize()
        assert torch.equal(c.view(torch.int16), want.view(torch.int16)), name
    assert not area[:4096].any() and B.axonn_linear_split_k_timeouts() == 0


@pytest.mark.gpu
@pytest.mark.parametrize("layout", LAYOUTS)
def test_ranges_that_do_not_wait_for_one_another(layout):
    """A range that looks once (0), a few times (3) or for long for the others of its tile: shares are handed on or not, with the same bits, the flags
    taken back, and in replays of a captured graph."""
    area = B.register_workspace()
    products = {name: shape for (name, lay), shape in eight_wave_split_products().items() if lay == layout}
    for name, (M, N, K) in sorted(products.items()):
        print(f"  {name} {layout} {(M, N, K)}", flush=True)
        x = torch.randn((K, M) if layout == "TN" else (M, K), device="cuda").to(torch.bfloat16)
        y = torch.randn((N, K) if layout == "NT" else (K, N), device="cuda").to(torch.bfloat16)
        want = torch.empty((M, N), dtype=torch.bfloat16, device="cuda")
        c = torch.empty_like(want)
        B.axonn_linear_gemm_split_probes(M, N, K, layout, x, y, want, 1 << 19)
        torch.cuda.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph):
            for _ in range(2):
                B.axonn_linear_gemm_split_probes(M, N, K, layout, x, y, c, 0)
        runs = [lambda p=p: B.axonn_linear_gemm_split_probes(M, N, K, layout, x, y, c, p) for p in (0, 0, 3)]
        for run in runs + [graph.replay] * 3 + [lambda: B.axonn_linear_fwd(M, N, K, layout, x, y, c)]:
            c.fill_(float("nan"))
            run()
            torch.cuda.synchronize()
            assert torch.equal(c.view(torch.int16), want.view(torch.int16)), name
            assert not area[:4096].any(), name


def test_the_entry_point_with_probes_refuses_other_kernels():
    at = 0x1000   # nothing is launched
    for args in ((256, 256, 256), (0, 256, 256)):
        with pytest.raises(B.AxonnError):
            B.axonn_linear_gemm_split_probes(*args, "NN", at, at, at, 0, stream=0)
    with pytest.raises(B.AxonnError):
        B.axonn_linear_gemm_split_probes(1024, 1024, 4096, "NT", at, at + 2, at, 0, stream=0)


@pytest.mark.gpu
def test_an_area_of_the_advertised_size_runs_the_planned_variant(oracle_mod):
    """The eight-wave kernel's partial sums take more than the variant's: without room for them the variant itself runs."""
    shape = (1024, 1024, 4096, "NT")
    B.register_workspace()
    wide = B.kernels(*shape, now=True)
    try:
        exact = torch.zeros((B.axonn_linear_workspace_bytes(*shape),), dtype=torch.uint8, device="cuda")
        B.axonn_linear_set_workspace(exact)
        assert B.kernels(*shape, now=True) == B.kernels(*shape) != wide
        _check(oracle_mod, *shape, B.kernels(*shape))
        assert not exact[:4096].any()
    finally:
        B.register_workspace()


@pytest.mark.gpu
def test_an_area_of_the_static_one_s_size_is_enough_for_the_eight_wave_kernel():
    B.register_workspace()
    products = [(*shape, layout) for (_, layout), shape in eight_wave_split_products().items()]
    rng = random.Random(19)   # large ones as well: names alone
    products += [(_log_int(rng, 128, 4096, 128), _log_int(rng, 128, 16384, 128), _log_int(rng, 512, 32000, 64), rng.choice(LAYOUTS)) for _ in range(2000)]
    wide = {p: B.kernels(*p, now=True) for p in products}
    try:
        need = max([B.axonn_linear_workspace_bytes(*p) for p in products] + [B.axonn_linear_static_scratch_bytes()])
        for size in (B.axonn_linear_static_scratch_bytes(), need):
            area = torch.zeros((size,), dtype=torch.uint8, device="cuda")
            B.axonn_linear_set_workspace(area)
            for p in products:
                if B.axonn_linear_workspace_bytes(*p) <= size:
                    assert B.kernels(*p, now=True) == wide[p], p
    finally:
        B.register_workspace()


@pytest.mark.gpu
def test_a_ragged_layer_s_data_gradient(oracle_mod):
    _check(oracle_mod, 1064, 1608, 4168, "NT", ["mfma16k64g_64x128_ktail"])


@pytest.mark.gpu
@pytest.mark.parametrize("shape", [(2048, 8192, 24), (1024, 4096, 32), (1025, 4099, 31), (600, 16384, 7), (3000, 5000, 1), (16384, 1024, 33),
                                   (2001, 8191, 63), (2000, 8200, 40), (65, 40001, 9), (4099, 2303, 63), (9000, 900, 8), (2048, 8192, 64),
                                   # one to three of a workgroup's four waves with columns of their own, in its first step or its last
                                   (65536, 64, 24), (65536, 64, 32), (40001, 65, 17), (20000, 128, 63), (16391, 192, 5), (16384, 257, 41), (60003, 320, 33),
                                   (9999, 520, 31), (30000, 576, 48), (48153, 392, 64), (43558, 208, 64),
                                   # rows off half lines from 8 MB on: another order of the workgroups (any number of them modulo 8)
                                   (2100, 2000, 24), (3301, 4099, 33), (8192, 1030, 7)])
def test_weight_gradient_of_a_few_tokens(oracle_mod, shape):
    """All of K in one chunk: K at the ends of the 8-row loads and of the 32-k halves, one step of columns a workgroup and two, ragged edges."""
    M, N, K = shape
    order = "_xcd" if N % 32 and M * N >= 4 << 20 else ""
    _check(oracle_mod, M, N, K, "TN", [f"wavek_64x64_k{32 if K <= 32 else 64}{order}"])


@pytest.mark.parametrize("shape", [(65536, 64, 48), (262144, 64, 64), (65536, 128, 64), (9200, 320, 64), (2001, 8191, 64),
                                   (18336, 21736, 8), (7688, 32056, 24)])
def test_weight_gradients_that_the_wave_k_kernel_does_faster(shape):
    """Narrow outputs over more than 32 k, rows off 128-byte lines over 64 and in large outputs: measured 0.58 to 0.95 times as fast on
    the other."""
    assert B.kernel_name(*shape, "TN") == "wavek_64x64_w1"


@pytest.mark.gpu
@pytest.mark.parametrize("layout", LAYOUTS)
@pytest.mark.parametrize("shape", [(300, 700, 5), (300, 700, 7), (515, 1031, 3), (2047, 2303, 4093), (3001, 1999, 2049)])
def test_guarded_kernel_on_misaligned_rows(oracle_mod, layout, shape):
    """Odd leading dimensions, several tiles, a ragged K: tiles moved back to the edge, whole pieces at any address."""
    edge = B.num_variants() - 1
    B.force_variant(edge)
    try:
        _check(oracle_mod, *shape, layout, ["edge_128x128"])
    finally:
        B.force_variant(-1)


@pytest.mark.gpu
@pytest.mark.parametrize("layout,shape", [("NN", (2048, 2056, 4096)), ("TN", (2048, 2056, 4096)), ("NT", (2048, 2056, 4096)),
                                          ("TN", (2056, 8192, 2048)), ("NN", (2049, 8192, 2048)), ("TN", (4104, 8200, 2048))])
def test_strips_narrower_than_sixteen(oracle_mod, layout, shape):
    """Strips of fewer than 16 rows or columns of an operand contiguous along them take the 16 last ones, some of which
    the launch over the whole tiles has written before."""
    B.register_workspace()
    M, N, K = shape
    kernels = B.kernels(M, N, K, layout)
    assert len(kernels) >= 2 and all(k.startswith("wavek") for k in kernels[1:]), kernels
    _check(oracle_mod, M, N, K, layout, kernels)


@pytest.mark.gpu
@pytest.mark.parametrize("layout,shape,kernel", [("NN", (1024, 3072, 3072), "mfma16k64g_128x128"), ("NT", (1024, 3072, 3072), "mfma16k64g_128x128"),
                                                 ("NN", (4099, 4099, 4099), "edge"), ("NN", (1000, 520, 1031), "wavek")])
def test_same_inputs_same_bits_on_the_kernel_named(layout, shape, kernel):
    B.register_workspace()
    M, N, K = shape
    assert B.kernel_name(M, N, K, layout, now=True).startswith(kernel)
    gen = torch.Generator(device="cuda").manual_seed(5)
    x = torch.randn((M, K), generator=gen, device="cuda").to(torch.bfloat16)
    y = torch.randn((N, K) if layout == "NT" else (K, N), generator=gen, device="cuda").to(torch.bfloat16)
    outs = [torch.empty((M, N), dtype=torch.bfloat16, device="cuda") for _ in range(3)]
    for c in outs[:2]:
        B.axonn_linear_fwd(M, N, K, layout, x, y, c)
    torch.cuda.synchronize()
    side = torch.cuda.Stream()
    with torch.cuda.stream(side):
        B.axonn_linear_fwd(M, N, K, layout, x, y, outs[2], stream=side)
    torch.cuda.synchronize()
    for c in outs[1:]:
        assert torch.equal(c.view(torch.int16), outs[0].view(torch.int16))
