"""GPU tests of single kernels and dispatch branches at the sizes where they can go wrong (edges of
tiles, remainders, the smallest and largest of a range), against the CPU oracle."""
import numpy as np
import pytest

from paper_2402_07710_amd import synth
from tests.test_gpu_parity import check_layer, say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("K,C_in,C_out", [(3, 256, 256), (3, 256, 80), (3, 128, 48), (3, 64, 16), (3, 32, 144), (5, 32, 32), (5, 64, 64),
                                          (5, 256, 16), (7, 32, 48)])
@pytest.mark.parametrize("n,dtype", [(1, "f16"), (65, "bf16"), (2000, "f16")])
def test_general_kernel(K, C_in, C_out, n, dtype):
    """Every number of input slices, output blocks that do and do not fill a workgroup's share, offsets
    beyond one mask word, and tiles with fewer offsets than a step holds."""
    say(f"general kernel K={K} {C_in}->{C_out} {dtype} n={n}")
    coords = synth.uniform_cells(n, 10 if n < 1000 else 20, seed=K + C_in + n)
    coords[:, 0] = np.arange(n) % 2
    check_layer(coords, K, 1, "subm", C_in, C_out, dtype, seed=n, out_dtype="f32" if n == 65 else None)


@pytest.mark.parametrize("K,C_in,dtype", [(7, 256, "f16"), (7, 64, "bf16"), (7, 32, "f16"), (5, 128, "f16"), (7, 16, "f32"), (3, 256, "f32"), (1, 64, "f16"), (3, 64, "bf16")])
@pytest.mark.parametrize("side", [1, 4, 9])
def test_general_kernel_on_a_cube(K, C_in, dtype, side):
    """Lists of offsets from one entry to all K^3 of them; with 256 input channels the list lies past 64 KB of LDS, in fp32
    an offset is up to four steps."""
    say(f"general kernel on a cube of {side}^3, K={K} C_in={C_in} {dtype}")
    xyz = np.stack(np.meshgrid(*[np.arange(side)] * 3, indexing="ij"), axis=-1).reshape(-1, 3)
    coords = np.concatenate([np.zeros((len(xyz), 1), dtype=np.int64), xyz], axis=1).astype(np.int32)
    check_layer(np.ascontiguousarray(coords), K, 1, "subm", C_in, 16 if C_in != 256 else 32, dtype, seed=side, threads=16)


def test_general_kernel_with_two_output_blocks_per_wavefront():
    say("general kernel, many tiles, 96 and 256 output channels")
    # up to 128 channels from four tiles per CU (of 256) on, 256 output channels from 0.75 on
    coords = np.concatenate([synth.lidar_scene(4)[:33000], synth.lidar_scene(5)[:33000]])
    coords[33000:, 0] = 1
    check_layer(coords, 3, 1, "subm", 32, 96, "f16", seed=1, threads=16)
    check_layer(coords[:13000], 3, 1, "subm", 32, 256, "bf16", seed=1, threads=16)


@pytest.mark.parametrize("K,stride,C_in,C_out", [(3, 1, 32, 64), (3, 1, 64, 64), (3, 1, 64, 128), (3, 1, 128, 128), (2, 2, 64, 128), (2, 2, 128, 128), (3, 2, 64, 64)])
@pytest.mark.parametrize("n,dtype", [(1, "bf16"), (64, "f16"), (129, "bf16"), (66000, "f16")])
def test_general_kernel_64_and_128_channels(K, stride, C_in, C_out, n, dtype):
    """One row, whole tiles, a tile of one row, and enough tiles for two output blocks per wavefront."""
    say(f"general kernel K={K} s={stride} {C_in}->{C_out} {dtype} n={n}")
    if n > 60000:
        coords = np.concatenate([synth.lidar_scene(4)[:33000], synth.lidar_scene(5)[:33000]])
        coords[33000:, 0] = 1
    else:
        coords = synth.uniform_cells(n, 9, seed=C_in + C_out + n)
    check_layer(coords, K, stride, "subm" if stride == 1 else "strided", C_in, C_out, dtype, seed=n, threads=16)


def test_streaming_kernel_strided_128_channels():
    """K = 2, 128 -> 128 beyond 20 tiles per CU (of 256), where the streaming kernel takes over; the last
    workgroup's eight tiles are not all there."""
    say("streaming kernel K=2 128->128")
    import oracle
    from tests.test_gpu_parity import rel_err, run_layer, sampled_rows_reference
    n = 350_000
    coords = synth.uniform_cells(n, 110, seed=2)
    feat, weight = synth.features(n, 128, "f16", 2), synth.weights(8, 128, 128, "f16", 2)
    _, h, out_coords, out = run_layer(coords, feat, weight, 2, 2, "strided", "f16", out_dtype="f32")
    km = oracle.kmap(coords, 2, 2, "strided")
    assert h.n_out == km["n_out"] and np.array_equal(out_coords, km["out_coords"])
    rows = np.unique(np.concatenate([np.random.default_rng(2).choice(h.n_out, 4000, replace=False), np.arange(200),
                                     np.arange(h.n_out - 200, h.n_out)]))
    err = rel_err(out[rows], sampled_rows_reference(feat, weight, km, rows)[rows])
    assert err <= 1e-5, err


@pytest.mark.parametrize("stride,n", [(1, 213_100), (2, 114_800)])
def test_streaming_kernel_32_to_64_channels(stride, n):
    """The fewest tiles that take it: 13 per CU (of 256), strided layers 7 (rows of the input)."""
    say(f"streaming kernel K=3 s={stride} 32->64")
    import oracle
    from tests.test_gpu_parity import rel_err, run_layer, sampled_rows_reference
    mode = "subm" if stride == 1 else "strided"
    coords = synth.uniform_cells(n, 90, seed=3)
    feat, weight = synth.features(n, 32, "f16", 3), synth.weights(27, 32, 64, "f16", 3)
    _, h, _, out = run_layer(coords, feat, weight, 3, stride, mode, "f16", out_dtype="f32")
    km = oracle.kmap(coords, 3, stride, mode)
    assert h.n_out == km["n_out"]
    rows = np.unique(np.concatenate([np.random.default_rng(3).choice(h.n_out, 4000, replace=False), np.arange(200),
                                     np.arange(h.n_out - 200, h.n_out)]))
    err = rel_err(out[rows], sampled_rows_reference(feat, weight, km, rows)[rows])
    assert err <= 1e-5, err


@pytest.mark.parametrize("K,stride,C,n", [(3, 1, 32, 147_457), (3, 2, 32, 147_457), (2, 2, 64, 147_457),
                                          (3, 2, 32, 32_640), (3, 2, 32, 32_705), (3, 2, 32, 64 * 512 + 1), (3, 2, 32, 64 * 1024), (3, 2, 32, 64 * 1024 + 1)])
def test_packed_square_layers_of_the_resident_kernel(K, stride, C, n):
    """Packed weights: 9 tiles per CU of 256 and one row more; strided layers up to 512 tiles and beyond 1,024, which take up to two tiles per
    workgroup, and between, up to four."""
    say(f"packed K={K} s={stride} {C}->{C} n={n}")
    import oracle
    import torch
    from paper_2402_07710_amd import binding as sc
    from tests.test_gpu_parity import rel_err, sampled_rows_reference, to_dev
    mode = "subm" if stride == 1 else "strided"
    coords = synth.uniform_cells(n, 80, seed=5)
    feat, weight = synth.features(n, C, "f16", 5), synth.weights(K ** 3, C, C, "f16", 5)
    buf = sc.LayerBuffers(n, K, stride, mode, C, C, "f16", out_dtype="f32", device="cuda:0")
    buf.feat_out.fill_(float("nan"))
    buf.hash_build(torch.from_numpy(coords).to("cuda:0"))
    buf.kmap_build(torch.from_numpy(coords).to("cuda:0"))
    buf.conv_fwd_packed(to_dev(feat, "f16"), sc.sc_conv_weight_pack(to_dev(weight, "f16"), K))
    km = oracle.kmap(coords, K, stride, mode)
    assert buf.read_counts().n_out == km["n_out"]
    rows = np.unique(np.concatenate([np.random.default_rng(5).choice(km["n_out"], 3000, replace=False), np.arange(200),
                                     np.arange(km["n_out"] - 200, km["n_out"])]))
    err = rel_err(buf.feat_out.cpu().numpy()[rows], sampled_rows_reference(feat, weight, km, rows)[rows])
    assert err <= 1e-5, err


@pytest.mark.parametrize("K,stride,C,n", [(3, 1, 32, 147_457), (3, 2, 32, 147_457), (2, 2, 64, 147_457),
                                          (3, 2, 32, 64 * 512), (3, 2, 32, 64 * 512 + 1), (3, 2, 32, 64 * 1024), (3, 2, 32, 64 * 1024 + 1)])
@pytest.mark.parametrize("dtype", ["f16", "bf16"])
def test_packed_and_raw_weights_agree_bit_for_bit(K, stride, C, n, dtype):
    """The resident kernel with packed weights and with raw ones, which it lays out itself: 9 tiles per CU (of 256) and more, and
    strided layers at the ends of the range that takes four tiles per workgroup."""
    say(f"packed and raw K={K} s={stride} {C}->{C} {dtype} n={n}")
    import torch
    from paper_2402_07710_amd import binding as sc
    from tests.test_gpu_parity import to_dev
    coords = torch.from_numpy(synth.uniform_cells(n, 80, seed=6)).to("cuda:0")
    feat, weight = to_dev(synth.features(n, C, dtype, 6), dtype), to_dev(synth.weights(K ** 3, C, C, dtype, 6), dtype)
    for out in (dtype, "f32"):
        buf = sc.LayerBuffers(n, K, stride, "subm" if stride == 1 else "strided", C, C, dtype, out_dtype=out, device="cuda:0")
        buf.hash_build(coords)
        buf.kmap_build(coords)
        buf.conv_fwd(feat, weight)
        raw = buf.feat_out[:buf.read_counts().n_out].clone()
        buf.feat_out.fill_(float("nan"))
        buf.conv_fwd_packed(feat, sc.sc_conv_weight_pack(weight, K))
        assert len(raw) > 1000 and torch.equal(buf.feat_out[:len(raw)], raw)


@pytest.mark.parametrize("C_in,C_out", [(32, 64), (64, 64), (64, 128), (128, 128)])
@pytest.mark.parametrize("n", [64, 129, 66000])
def test_fused_general_kernel(C_in, C_out, n):
    """Look-ups inside the general kernel: a workgroup's tile is full, has one row, and two output blocks per
    wavefront; voxels on the faces of the box."""
    say(f"fused general kernel {C_in}->{C_out} n={n}")
    import oracle
    import torch
    from paper_2402_07710_amd import binding as sc
    from tests.test_gpu_parity import TOL, rel_err, to_dev
    side = 10 if n < 1000 else 50
    coords = synth.uniform_cells(n, side, seed=n)
    feat, weight = synth.features(n, C_in, "f16", 1), synth.weights(27, C_in, C_out, "f16", 1)
    buf = sc.LayerBuffers(n, 3, 1, "subm", C_in, C_out, "f16", device="cuda:0", grid_dims=(1, side, side, side))
    buf.feat_out.fill_(float("nan"))
    buf.layer_fused(torch.from_numpy(coords).to("cuda:0"), to_dev(feat, "f16"), to_dev(weight, "f16"))
    ref = oracle.conv(feat, weight, oracle.kmap(coords, 3, 1, "subm"), threads=16)
    err = rel_err(buf.feat_out[:n].double().cpu().numpy(), ref)
    assert err <= TOL["f16"], err


@pytest.mark.parametrize("K,C_in,C_out,n", [(3, 16, 64, 17000), (3, 32, 32, 17000), (3, 64, 64, 1), (3, 64, 64, 65), (3, 64, 80, 1000),
                                            (3, 128, 16, 700), (3, 256, 48, 300), (5, 16, 16, 700), (5, 32, 32, 65), (1, 16, 80, 17000), (1, 64, 16, 24500),
                                            (3, 16, 64, 24500), (3, 32, 32, 16400), (3, 64, 64, 34000), (3, 64, 80, 5000),
                                            (3, 128, 64, 5000), (3, 256, 48, 8000), (5, 32, 32, 30000)])
def test_general_kernel_fp32(K, C_in, C_out, n):
    """fp32: weights through LDS, rows of one to sixteen slices; 16 channels per workgroup of four wavefronts (the
    first two rows of the list) and, where the last round of the 256 CUs is no shorter with 16, 32 per workgroup
    of eight (the others), also with a last block that is not there (80, 48)."""
    say(f"general kernel fp32 K={K} {C_in}->{C_out} n={n}")
    coords = synth.lidar_scene(3)[:n] if n > 2000 else synth.uniform_cells(n, 10, seed=K + C_in + n)
    check_layer(coords, K, 1, "subm", C_in, C_out, "f32", seed=n, threads=16)


@pytest.mark.parametrize("C_in,C_out", [(16, 64), (32, 32), (64, 16), (32, 48), (16, 80)])
@pytest.mark.parametrize("n", [1900, 4000, 17000])
def test_strided_fp32_on_both_sides_of_the_line(C_in, C_out, n):
    """fp32 layers of 1,024 to 2,047 channel products, K = 3, stride 2: bound and expected tiles on either side of
    a tile per CU (of 256)."""
    say(f"strided fp32 {C_in}->{C_out} n={n}")
    check_layer(synth.lidar_scene(6)[:n], 3, 2, "strided", C_in, C_out, "f32", seed=n, threads=16)


@pytest.mark.parametrize("K,stride,C_in,C_out", [(3, 1, 1, 16), (3, 1, 3, 64), (3, 1, 4, 32), (2, 2, 4, 16), (2, 2, 3, 32), (2, 2, 2, 64)])
@pytest.mark.parametrize("n", [1, 64, 65, 3000])
def test_first_layer_fp32(K, stride, C_in, C_out, n):
    """At most four input channels: rows and weights short of four, tiles that are full and that have one row."""
    say(f"first layer K={K} s={stride} {C_in}->{C_out} n={n}")
    coords = synth.uniform_cells(n, 6 if n < 100 else 18, seed=C_in + n)
    check_layer(coords, K, stride, "subm" if stride == 1 else "strided", C_in, C_out, "f32", seed=n)


@pytest.mark.parametrize("K,stride", [(2, 2), (3, 2), (3, 3), (4, 2), (5, 5)])
@pytest.mark.parametrize("n", [1, 256, 257, 3000])
def test_strided_build_claims(K, stride, n):
    """The merged claims of output cells at the edges of a workgroup, for the compiled-in shapes and the
    general one, on sets where many inputs share a cell (a full cube) and where none do (a lattice)."""
    say(f"strided claims K={K} s={stride} n={n}")
    side = int(np.ceil(n ** (1 / 3)))
    cube = np.stack(np.meshgrid(*[np.arange(side)] * 3, indexing="ij"), axis=-1).reshape(-1, 3)[:n]
    for xyz in (cube, cube * 8 + 7):
        coords = np.concatenate([np.arange(len(xyz))[:, None] % 2, xyz], axis=1).astype(np.int32)
        check_layer(np.ascontiguousarray(coords), K, stride, "strided", 32, 32, "f16", seed=n)


def test_strided_map_with_blocks_of_4096_candidates():
    say("strided map, 560,000 and 4.5 M candidates")
    from paper_2402_07710_amd import binding as sc
    import oracle
    import torch
    from tests.test_gpu_parity import assert_maps_equal, exported_map
    for n, K in ((70_000, 3), (560_000, 3), (600_000, 2)):
        coords = synth.uniform_cells(n, 100, seed=n)
        buf = sc.LayerBuffers(n, K, 2, "strided", 32, 32, "f16", device="cuda:0")
        buf.kmap_build(torch.from_numpy(coords).to("cuda:0"), standalone=True)
        h = buf.read_counts()
        ref = oracle.kmap(coords, K, 2, "strided")
        assert h.status == 0 and h.n_out == ref["n_out"] and h.n_pairs == ref["offset_start"][-1]
        assert_maps_equal(exported_map(buf, h), buf.out_coords[:h.n_out].cpu().numpy(), ref, exact_order=True)


@pytest.mark.parametrize("K", [3, 5])
@pytest.mark.parametrize("n", [1, 65, 3000, 270_000])
def test_submanifold_map_lookups(K, n):
    """The look-ups of a submanifold map by block: sets at the ends of the coordinate domain, cubes that
    cross every block boundary, and enough rows for the variant with one wavefront per x offset."""
    say(f"submanifold look-ups K={K} n={n}")
    from paper_2402_07710_amd import binding as sc
    import oracle
    import torch
    from tests.test_gpu_parity import assert_maps_equal, exported_map
    cells = synth.uniform_cells(n, 16 if n <= 3000 else 90, seed=K + n)
    for base in (0, sc.SC_COORD_MAX - int(cells[:, 1:].max())):
        coords = cells.copy()
        coords[:, 0] = np.arange(n) % 2 * 255 if n <= 3000 else 3
        coords[:, 1:] += base
        buf = sc.LayerBuffers(n, K, 1, "subm", 32, 32, "f16", device="cuda:0")
        dev = torch.from_numpy(coords).to("cuda:0")
        buf.hash_build(dev)
        buf.kmap_build(dev)
        h = buf.read_counts()
        ref = oracle.kmap(coords, K, 1, "subm")
        assert h.status == 0 and h.n_out == n
        assert_maps_equal(exported_map(buf, h), coords, ref, exact_order=True)
        if n > 3000:
            break


@pytest.mark.parametrize("K,C_in,C_out,dtype", [(5, 32, 32, "f16"), (5, 32, 48, "bf16"), (7, 32, 32, "f16"), (3, 32, 16, "f16"), (3, 32, 64, "f16"),
                                                (3, 32, 144, "bf16"), (3, 32, 32, "f16"), (3, 64, 64, "f16"), (3, 128, 128, "bf16"),
                                                (3, 256, 32, "f16"), (3, 32, 64, "f32"), (3, 16, 16, "f32"), (3, 4, 16, "f32")])
def test_non_finite_weights_stay_in_their_groups(K, C_in, C_out, dtype):
    """An infinite W[k] reaches the 16-row groups that have a neighbour at k, and no others: the same
    bits there as without it, also in tiles whose other groups do have one."""
    say(f"non-finite weights K={K} {C_in}->{C_out} {dtype}")
    import oracle
    import torch
    from tests.test_gpu_parity import run_layer
    n, K3 = 500, K ** 3
    coords = synth.uniform_cells(n, 30, seed=K)
    km = oracle.kmap(coords, K, 1, "subm")
    feat, weight = synth.features(n, C_in, dtype, 2), synth.weights(K3, C_in, C_out, dtype, 2)
    plain = run_layer(coords, feat, weight, K, 1, "subm", dtype)[3]
    start = km["offset_start"]
    has = np.zeros((K3, (n + 15) // 16), dtype=bool)           # [offset, group]
    for k in range(K3):
        has[k, km["pair_out"][start[k]:start[k + 1]] // 16] = True
    mixed = [k for k in range(K3) if has[k].any() and not has[k].all()]
    for k in mixed[::max(1, len(mixed) // 4)]:
        for value in (np.inf, np.nan):
            spoiled = weight.copy()
            spoiled[k] = value
            got = run_layer(coords, feat, spoiled, K, 1, "subm", dtype)[3]
            outside = ~has[k][np.arange(n) // 16]
            tiles = np.arange(n)[outside] // 64
            assert any(has[k][4 * t:4 * t + 4].any() for t in tiles), "a tile with and without"
            assert np.array_equal(got[outside], plain[outside]), k
            pair_rows = np.unique(km["pair_out"][start[k]:start[k + 1]])
            assert not np.isfinite(got[pair_rows]).all(axis=1).any()


@pytest.mark.parametrize("K", [2, 3, 4])
@pytest.mark.parametrize("stale", ["inverse map", "zeros", "ones", "words of the rows", "words of other rows"])
def test_inverse_map_of_rows_without_a_parent(K, stale):
    """Rows outside the coordinate domain have no parent, so their place in the inverse map's buffer is never
    written with one: whatever an earlier use left there must not become a pair."""
    say(f"inverse map, rows without a parent, K={K}, buffer holds {stale}")
    import oracle
    import torch
    from paper_2402_07710_amd import binding as sc
    from tests.test_gpu_parity import TOL, rel_err, to_dev
    n, K3 = 1000, K ** 3
    coords = synth.uniform_cells(n, 30, seed=K)
    out_of_domain = np.arange(n) % 7 == 3
    out_of_domain[640:704] = True                              # a whole tile of the fine rows
    broken = coords.copy()
    broken[out_of_domain, 1] = sc.SC_COORD_MAX + 1

    def inverse(rows, into):
        buf = sc.LayerBuffers(n, K, K, "strided", 32, 32, "f16", device="cuda:0")
        buf.kmap_build(torch.from_numpy(rows).to("cuda:0"), standalone=True)
        h = buf.read_counts(check=False)
        sc.sc_kmap_transpose(buf.kmap, n, K, K, buf.counts, into)
        return buf, h
    tiles, words = (n + 63) // 64, 4 * ((K3 + 31) // 32)
    first_line = (256 + tiles * words * 4 + 255) // 256 * 256 // 4          # int32 index of row 0's entry at offset 0
    into = torch.zeros(sc.sc_kmap_bytes(n, K, K, "inverse"), dtype=torch.uint8, device="cuda:0")
    if stale == "ones":
        into.fill_(255)
    elif stale != "zeros":
        _, h = inverse(coords, into)
        assert h.status == 0
        if stale != "inverse map":                             # (parent, offset) of every row as the first kernel writes it
            km = oracle.kmap(coords, K, K, "strided")
            word = np.zeros(n, dtype=np.int32)
            word[km["pair_in"]] = km["pair_out"] * 64 + np.repeat(np.arange(K3), np.diff(km["offset_start"]))
            if stale == "words of other rows":
                word = np.roll(word, 1)
            at = first_line + np.arange(n) // 64 * (K3 * 64) + np.arange(n) % 64
            into.view(torch.int32)[torch.from_numpy(at).to("cuda:0")] = torch.from_numpy(word).to("cuda:0")
    buf, h = inverse(broken, into)
    assert h.status == sc.SC_ERANGE
    kept = np.flatnonzero(~out_of_domain)
    ref = oracle.transpose_map(oracle.kmap(coords[kept], K, K, "strided"))
    h = sc.sc_counts_read(buf.counts, into, n, K, K, "inverse", check=False)
    assert h.n_pairs == len(kept) and list(h.per_offset[:K3]) == list(np.diff(ref["offset_start"]))
    pin, pout, _ = sc.sc_kmap_export(into, n, K, K, "inverse", h)
    assert np.array_equal(pin.cpu().numpy(), ref["pair_in"]) and np.array_equal(pout.cpu().numpy(), kept[ref["pair_out"]])
    # and the group masks: rows without a parent become zero, the others their products
    feat, weight = synth.features(int(ref["n_in"]), 32, "f16", K), synth.weights(K3, 32, 32, "f16", K)
    out = torch.full((n, 32), float("nan"), dtype=torch.float16, device="cuda:0")
    ws = torch.empty(sc.sc_conv_workspace_bytes(K, 32, 32, "f16"), dtype=torch.uint8, device="cuda:0")
    sc.sc_conv_fwd(to_dev(feat, "f16"), to_dev(weight, "f16"), out, into, buf.counts, K, K, "inverse", ws, n_map=n)
    got = out.double().cpu().numpy()
    assert np.all(got[out_of_domain] == 0)
    assert rel_err(got[kept], oracle.conv(feat, weight, ref, threads=8)) <= TOL["f16"]


@pytest.mark.parametrize("K,C_in,C_out,dtype", [(3, 3, 16, "f32"), (3, 5, 7, "f32"), (3, 16, 32, "f32"), (3, 64, 64, "f32"), (3, 32, 32, "f16"), (3, 32, 80, "bf16"),
                                                (3, 128, 64, "f16"), (2, 5, 20, "f32"), (2, 32, 16, "f32"), (2, 128, 32, "f32"), (2, 32, 64, "f16"), (2, 256, 48, "bf16"),
                                                (4, 64, 32, "f16"), (4, 16, 64, "f32")])
@pytest.mark.parametrize("n", [1, 65, 1500])
def test_strided_maps_with_and_without_masks(K, C_in, C_out, dtype, n):
    """K <= 3: every kernel votes over the map's lines, also those of a last tile that is not full; K = 4: masks of two words."""
    say(f"strided K={K} {C_in}->{C_out} {dtype} n={n}")
    check_layer(synth.uniform_cells(n, 6 if n < 100 else 14, seed=C_in + n), K, 2, "strided", C_in, C_out, dtype, seed=n)


@pytest.mark.parametrize("K,n", [(K, n) for K in (2, 3, 4) for n in (1, 64, 700, 5000)] + [(2, 262145), (3, 155329)])
def test_inverse_map_of_repeated_coordinates(K, n):
    """A build without a location table takes repeated inputs: one of them is in the map, and the inverse map holds the same pairs.
    The two largest sets take the longer build."""
    say(f"inverse map of repeated coordinates K={K} n={n}")
    import torch
    from paper_2402_07710_amd import binding as sc
    coords = synth.uniform_cells(n, 24 if n < 10000 else 90, seed=n)
    coords[n // 2:] = coords[:n - n // 2]
    buf = sc.LayerBuffers(n, K, K, "strided", 32, 32, "f16", device="cuda:0")
    buf.kmap_build(torch.from_numpy(np.ascontiguousarray(coords)).to("cuda:0"), standalone=True)
    h = buf.read_counts()
    pin, pout, _ = (t.cpu().numpy() for t in buf.export(h))
    into = torch.full((sc.sc_kmap_bytes(n, K, K, "inverse"),), 7, dtype=torch.uint8, device="cuda:0")
    sc.sc_kmap_transpose(buf.kmap, n, K, K, buf.counts, into)
    hi = sc.sc_counts_read(buf.counts, into, n, K, K, "inverse")
    iin, iout, _ = (t.cpu().numpy() for t in sc.sc_kmap_export(into, n, K, K, "inverse", hi))
    assert h.n_pairs == hi.n_pairs == len(np.unique(coords, axis=0)) and list(h.per_offset[:K ** 3]) == list(hi.per_offset[:K ** 3])
    offset = np.repeat(np.arange(K ** 3), h.per_offset[:K ** 3])
    assert sorted(zip(offset, pout, pin)) == sorted(zip(offset, iin, iout))


@pytest.mark.parametrize("K,n", [(2, 1), (2, 63), (2, 1024), (2, 1025), (2, 262144), (2, 262145), (3, 155328), (3, 155329), (4, 65536), (4, 65537), (5, 16768), (5, 16769), (5, 33536), (6, 9664), (6, 9665), (7, 6080),
                                 (7, 6081), (7, 12224)])
def test_strided_build_on_both_sides_of_the_short_one(K, n):
    """K == stride: cells with one input and with many, in random order; the largest sets whose words are counted by every
    workgroup or whose table is cleared ahead, and one row more."""
    say(f"strided build K=s={K} n={n}")
    import oracle
    import torch
    from paper_2402_07710_amd import binding as sc
    coords = synth.uniform_cells(n, max(4, int(round((n * 3) ** (1 / 3)))), seed=K + n)
    km = oracle.kmap(coords, K, K, "strided")
    buf = sc.LayerBuffers(n, K, K, "strided", 32, 32, "f16", device="cuda:0")
    buf.scratch.fill_(0x5a)
    buf.kmap.fill_(0x11)
    buf.kmap_build(torch.from_numpy(coords).to("cuda:0"), standalone=True)
    h = buf.read_counts()
    pin, pout, start = (t.cpu().numpy() for t in buf.export(h))
    assert h.n_out == km["n_out"] and np.array_equal(start, km["offset_start"])
    assert np.array_equal(pin, km["pair_in"]) and np.array_equal(pout, km["pair_out"])
    assert np.array_equal(buf.out_coords[:h.n_out].cpu().numpy(), km["out_coords"])


@pytest.mark.parametrize("K,n", [(3, 1536 * 64), (3, 1536 * 64 + 1), (3, 2300 * 64), (3, 2300 * 64 + 1), (3, 2304 * 64 + 63), (5, 896 * 64),
                                 (5, 896 * 64 + 1), (5, 1400 * 64 + 1)])
def test_map_of_tiles_in_runs(K, n):
    """The most tiles that go to the XCDs in eighths, the fewest that go in runs (6 and 3.5 per CU of 256), last runs that are not full."""
    say(f"map in runs K={K} n={n}")
    import oracle
    import torch
    from paper_2402_07710_amd import binding as sc
    coords = synth.uniform_cells(n, 64, seed=K)
    km = oracle.kmap(coords, K, 1, "subm")
    buf = sc.LayerBuffers(n, K, 1, "subm", 32, 32, "f16", device="cuda:0")
    c = torch.from_numpy(coords).to("cuda:0")
    buf.kmap.fill_(0x11)
    buf.hash_build(c)
    buf.kmap_build(c)
    pin, pout, start = (t.cpu().numpy() for t in buf.export())
    assert np.array_equal(start, km["offset_start"]) and np.array_equal(pin, km["pair_in"]) and np.array_equal(pout, km["pair_out"])


@pytest.mark.parametrize("C_out,n", [(64, 768 * 64), (64, 768 * 64 + 1), (128, 384 * 64), (128, 384 * 64 + 1), (16, 33), (256, 193 * 64)])
def test_64_channel_steps_on_both_sides_of_three_workgroups_per_cu(C_out, n):
    """Steps of two offsets, with an odd number of offsets in a tile's list, and of one; with and without a map."""
    say(f"64 -> {C_out}, n={n}")
    import torch
    from paper_2402_07710_amd import binding as sc
    from tests.test_gpu_parity import TOL, to_dev
    side = max(4, int(round((n * 3) ** (1 / 3))))
    coords = synth.uniform_cells(n, side, seed=C_out)
    feat, weight = synth.features(n, 64, "bf16", 1), synth.weights(27, 64, C_out, "bf16", 1)
    buf = sc.LayerBuffers(n, 3, 1, "subm", 64, C_out, "bf16", device="cuda:0")
    c, f, w = torch.from_numpy(coords).to("cuda:0"), to_dev(feat, "bf16"), to_dev(weight, "bf16")
    buf.feat_out.fill_(float("nan"))
    buf.layer(c, f, w)
    pin, pout, start = (t.long() for t in buf.export())
    ref = torch.zeros((n, C_out), device="cuda:0")
    for k in range(27):
        at = slice(int(start[k]), int(start[k + 1]))
        ref.index_add_(0, pout[at], f[pin[at]].float() @ w[k].float())
    assert float((buf.feat_out.float() - ref).abs().max() / ref.abs().max()) <= TOL["bf16"]
    if C_out in (64, 128):
        fused = sc.LayerBuffers(n, 3, 1, "subm", 64, C_out, "bf16", device="cuda:0", grid_dims=(1, side, side, side))
        fused.layer_fused(c, f, w)
        assert torch.equal(fused.feat_out, buf.feat_out)


@pytest.mark.parametrize("K,n", [(2, 262145), (3, 155329), (4, 65537), (5, 16769), (5, 33000), (6, 9665), (7, 6081)])
def test_large_tables_are_cleared_where_rows_exist(K, n):
    """K == stride: of a table that is more than a build should clear ahead, the rows that no cell has stay as they were."""
    say(f"rows that do not exist K=s={K} n={n}")
    import oracle
    import torch
    from paper_2402_07710_amd import binding as sc
    coords = synth.lidar_scene(1)
    coords = np.ascontiguousarray(np.concatenate([np.concatenate([np.full((len(coords), 1), b), coords[:, 1:]], axis=1) for b in range(5)])[:n].astype(np.int32))
    buf = sc.LayerBuffers(n, K, K, "strided", 32, 32, "f16", device="cuda:0")
    buf.kmap.fill_(0x11)
    buf.kmap_build(torch.from_numpy(coords).to("cuda:0"), standalone=True)
    n_out = buf.read_counts().n_out
    assert n_out == oracle.kmap(coords, K, K, "strided")["n_out"] < n
    K3, tiles, used = K ** 3, (n + 63) // 64, (n_out + 63) // 64
    first = (256 + tiles * 16 * ((K3 + 31) // 32) + 255) // 256 * 256 // 4       # int32 index of the table
    table = buf.kmap[:(first + tiles * K3 * 64) * 4].view(torch.int32)[first:].view(tiles, K3 * 64)
    assert used < tiles and bool((table[used:] == 0x11111111).all())
    assert not bool((table[:used] == 0x11111111).any())


@pytest.mark.parametrize("stride,C_in,C_out,n", [(2, 128, 128, 393_217), (3, 128, 128, 400_000), (2, 32, 64, 400_000)])
def test_streaming_kernel_strided_rows_known_to_the_caller(stride, C_in, C_out, n):
    """K = 3, the output holds exactly the rows there are.  128 -> 128: strided layers of inputs that would leave a round part-filled;
    32 -> 64: stride 2, rows between 7 and 13 tiles per CU (of 256)."""
    say(f"streaming kernel K=3 s={stride} {C_in}->{C_out} n={n}")
    import oracle
    import torch
    from paper_2402_07710_amd import binding as sc
    from tests.test_gpu_parity import rel_err, sampled_rows_reference, to_dev
    coords = synth.uniform_cells(n, 80 if C_in == 128 else 110, seed=stride)
    feat, weight = synth.features(n, C_in, "f16", 3), synth.weights(27, C_in, C_out, "f16", 3)
    buf = sc.LayerBuffers(n, 3, stride, "strided", 32, 32, "f16", device="cuda:0")
    buf.kmap_build(torch.from_numpy(coords).to("cuda:0"), standalone=True)
    km = oracle.kmap(coords, 3, stride, "strided")
    n_out = buf.read_counts().n_out
    assert n_out == km["n_out"]
    assert C_in == 128 or 7 * 256 < n_out / 64 <= 13 * 256
    out = torch.full((n_out, C_out), float("nan"), dtype=torch.float32, device="cuda:0")
    packed = sc.sc_conv_weight_pack(to_dev(weight, "f16"), 3)
    sc.sc_conv_fwd_packed(to_dev(feat, "f16"), packed, C_out, out, buf.kmap, buf.counts, 3, stride, "strided", n_map=n)
    rows = np.unique(np.concatenate([np.random.default_rng(3).choice(n_out, 3000, replace=False), np.arange(200), np.arange(n_out - 200, n_out)]))
    err = rel_err(out.cpu().numpy()[rows], sampled_rows_reference(feat, weight, km, rows)[rows])
    assert err <= 1e-5, err


@pytest.mark.parametrize("n", [400_000, 436_864, 436_865])
def test_128_channels_on_both_sides_of_rounds_five_sixths_full(n):
    """K = 3, 24 to 26 2/3 tiles per CU (of 256) and one tile more, with a map and fused."""
    say(f"128 -> 128, n={n}")
    import torch
    from paper_2402_07710_amd import binding as sc
    from tests.test_gpu_parity import to_dev
    coords = synth.uniform_cells(n, 110, seed=n)
    feat, weight = synth.features(n, 128, "f16", 1), synth.weights(27, 128, 128, "f16", 1)
    buf = sc.LayerBuffers(n, 3, 1, "subm", 128, 128, "f16", out_dtype="f32", device="cuda:0")
    c, f, w = torch.from_numpy(coords).to("cuda:0"), to_dev(feat, "f16"), to_dev(weight, "f16")
    buf.feat_out.fill_(float("nan"))
    buf.layer(c, f, w)
    pin, pout, start = (t.long() for t in buf.export())
    ref = torch.zeros((n, 128), device="cuda:0")
    for k in range(27):
        at = slice(int(start[k]), int(start[k + 1]))
        ref.index_add_(0, pout[at], f[pin[at]].float() @ w[k].float())
    assert float((buf.feat_out - ref).abs().max() / ref.abs().max()) <= 1e-5
    fused = sc.LayerBuffers(n, 3, 1, "subm", 128, 128, "f16", out_dtype="f32", device="cuda:0", grid_dims=(1, 110, 110, 110))
    fused.feat_out.fill_(float("nan"))
    fused.layer_fused(c, f, w)
    assert float((fused.feat_out - ref).abs().max() / ref.abs().max()) <= 1e-5


@pytest.mark.parametrize("C_out,n", [(64, 512 * 64 + 1), (64, 768 * 64), (64, 768 * 64 + 1), (128, 384 * 64), (128, 384 * 64 + 1), (16, 33)])
def test_32_channel_steps_on_both_sides_of_three_workgroups_per_cu(C_out, n):
    """Steps of four offsets, with lists that do not fill the last one, and of two; with and without a map."""
    say(f"32 -> {C_out}, n={n}")
    import torch
    from paper_2402_07710_amd import binding as sc
    from tests.test_gpu_parity import TOL, to_dev
    side = max(4, int(round((n * 3) ** (1 / 3))))
    coords = synth.uniform_cells(n, side, seed=C_out)
    feat, weight = synth.features(n, 32, "f16", 1), synth.weights(27, 32, C_out, "f16", 1)
    buf = sc.LayerBuffers(n, 3, 1, "subm", 32, C_out, "f16", device="cuda:0")
    c, f, w = torch.from_numpy(coords).to("cuda:0"), to_dev(feat, "f16"), to_dev(weight, "f16")
    buf.feat_out.fill_(float("nan"))
    buf.layer(c, f, w)
    pin, pout, start = (t.long() for t in buf.export())
    ref = torch.zeros((n, C_out), device="cuda:0")
    for k in range(27):
        at = slice(int(start[k]), int(start[k + 1]))
        ref.index_add_(0, pout[at], f[pin[at]].float() @ w[k].float())
    assert float((buf.feat_out.float() - ref).abs().max() / ref.abs().max()) <= TOL["f16"]
    if C_out == 64:
        fused = sc.LayerBuffers(n, 3, 1, "subm", 32, C_out, "f16", device="cuda:0", grid_dims=(1, side, side, side))
        fused.layer_fused(c, f, w)
        assert torch.equal(fused.feat_out, buf.feat_out)


@pytest.mark.parametrize("K,stride,C_in,C_out,n", [(5, 1, 128, 256, 832 * 64), (5, 1, 128, 256, 832 * 64 + 1), (5, 1, 64, 256, 832 * 64 + 1), (5, 1, 256, 240, 900 * 64 - 7),
                                                   (7, 1, 64, 256, 833 * 64), (4, 2, 256, 256, 60_000), (7, 1, 128, 256, 576 * 64),
                                                   (7, 1, 128, 256, 576 * 64 + 1), (6, 3, 256, 256, 8502), (6, 3, 256, 112, 9000), (7, 3, 128, 240, 8502)])
def test_blocks_of_output_channels_together_and_apart(K, stride, C_in, C_out, n):
    """16 bit, two to four blocks per tile, on both sides of 3 1/4 and 2 1/4 tiles per CU (of 256) and of 6 and 12 MiB of weights; a last block that is
    not full, and tiles that are known on the device only, several times the inputs' (K = 6 and 7 with stride 3)."""
    say(f"blocks apart K={K} s={stride} {C_in}->{C_out} n={n}")
    import torch
    from paper_2402_07710_amd import binding as sc
    from tests.test_gpu_parity import to_dev
    coords = synth.uniform_cells(n, 200 if stride == 3 else 100, seed=K)
    feat, weight = synth.features(n, C_in, "f16", 1), synth.weights(K ** 3, C_in, C_out, "f16", 1)
    buf = sc.LayerBuffers(n, K, stride, "subm" if stride == 1 else "strided", C_in, C_out, "f16", out_dtype="f32", device="cuda:0")
    c, f, w = torch.from_numpy(coords).to("cuda:0"), to_dev(feat, "f16"), to_dev(weight, "f16")
    buf.feat_out.fill_(float("nan"))
    buf.layer(c, f, w)
    n_out = buf.read_counts().n_out
    assert stride == 1 or n_out > 833 * 64
    pin, pout, start = (t.long() for t in buf.export())
    ref = torch.zeros((n_out, C_out), device="cuda:0")
    for k in range(K ** 3):
        at = slice(int(start[k]), int(start[k + 1]))
        ref.index_add_(0, pout[at], f[pin[at]].float() @ w[k].float())
    assert float((buf.feat_out[:n_out] - ref).abs().max() / ref.abs().max()) <= 1e-5
    assert bool(buf.feat_out[n_out:].isnan().all())


@pytest.mark.parametrize("K,stride,C_in,C_out,n,grid", [(7, 1, 16, 16, 896 * 64, 40), (7, 1, 16, 16, 896 * 64 + 1, 40), (7, 1, 32, 16, 62_000, 120), (5, 1, 16, 16, 1024 * 64, 41),
                                                        (5, 1, 64, 16, 1024 * 64 + 1, 41), (5, 1, 128, 16, 60_000, 60), (4, 1, 256, 16, 60_000, 50), (6, 2, 16, 16, 60_000, 60),
                                                        (4, 4, 16, 16, 62_000, 60)])
def test_list_of_offsets_in_registers(K, stride, C_in, C_out, n, grid):
    """fp32, 16 output channels, K >= 4, on both sides of 3 1/2 and of 4 tiles per CU (of 256): tiles that take part in all of 343 offsets (the list goes on
    in the next register every 64), in few, rows of more than one step; K > stride, and K == stride."""
    say(f"list in registers K={K} s={stride} {C_in}->{C_out} n={n}")
    import torch
    from paper_2402_07710_amd import binding as sc
    from tests.test_gpu_parity import to_dev
    coords = synth.uniform_cells(n, grid, seed=K)
    feat, weight = synth.features(n, C_in, "f32", 1), synth.weights(K ** 3, C_in, C_out, "f32", 1)
    buf = sc.LayerBuffers(n, K, stride, "subm" if K % 2 else "strided", C_in, C_out, "f32", device="cuda:0")
    c, f, w = torch.from_numpy(coords).to("cuda:0"), to_dev(feat, "f32"), to_dev(weight, "f32")
    buf.feat_out.fill_(float("nan"))
    buf.layer(c, f, w)
    n_out = buf.read_counts().n_out
    pin, pout, start = (t.long() for t in buf.export())
    ref = torch.zeros((n_out, C_out), dtype=torch.float64, device="cuda:0")
    for k in range(K ** 3):
        at = slice(int(start[k]), int(start[k + 1]))
        ref.index_add_(0, pout[at], f[pin[at]].double() @ w[k].double())
    assert float((buf.feat_out[:n_out] - ref).abs().max() / ref.abs().max()) <= 1e-5
    assert bool(buf.feat_out[n_out:].isnan().all())


@pytest.mark.parametrize("C_in,C_out", [(32, 64), (64, 64), (64, 128), (128, 16), (256, 48)])
@pytest.mark.parametrize("n,dtype", [(1, "f16"), (64, "bf16"), (65, "f16"), (34000, "f16"), (1, "f32"), (65, "f32"), (17000, "f32")])
def test_pointwise_layers(C_in, C_out, n, dtype):
    """K = 1: a list of one offset, read from the map; whole tiles, a tile of one row, and two output blocks per wavefront (64 -> 128); in
    fp32 a row of 128 and more channels is more than one step."""
    say(f"K=1 {C_in}->{C_out} {dtype} n={n}")
    if n < 1000:
        coords = synth.uniform_cells(n, 6, seed=n)
    else:
        coords = np.concatenate([synth.lidar_scene(4)[:n], synth.lidar_scene(5)[:n]])
        coords[n:, 0] = 1
    check_layer(np.ascontiguousarray(coords), 1, 1, "subm", C_in, C_out, dtype, seed=n, threads=16)


def test_more_workgroups_than_a_row_of_the_grid_holds():
    """fp32, 240 output channels, room for SC_N_MAX rows: 2^20 tiles of 8 blocks of output channels, 2^23 workgroups of 512 threads.
    A full 256 x 256 x 128 box, K = 3, stride 2: cell q has the inputs 2 q + d inside the box."""
    say("2^26 rows of 240 channels")
    import torch
    from paper_2402_07710_amd import binding as sc
    dev, X, Y, Z, C_in, C_out = "cuda:0", 256, 256, 128, 16, 240
    n = X * Y * Z
    lin = torch.arange(n, device=dev)
    coords = torch.stack([torch.zeros_like(lin), lin // (Y * Z), lin // Z % Y, lin % Z], dim=1).int().contiguous()
    feat = (lin[:, None] * 2654435761 + torch.arange(C_in, device=dev) * 40503).remainder(4093).float() / 2048 - 1
    weight = torch.from_numpy(synth.weights(27, C_in, C_out, "f32", 9)).to(dev)
    buf = sc.LayerBuffers(n, 3, 2, "strided", C_in, C_out, "f32", device=dev)
    assert buf.feat_out.shape[0] == 1 << 26
    buf.kmap_build(coords, standalone=True)
    n_out = X // 2 * (Y // 2) * (Z // 2)
    buf.feat_out[:n_out + 64] = float("nan")
    buf.conv_fwd(feat, weight)
    assert buf.read_counts().n_out == n_out
    assert not bool(buf.feat_out[:n_out].isnan().any()) and bool(buf.feat_out[n_out:n_out + 64].isnan().all())
    rows = torch.cat([torch.arange(128, device=dev), torch.arange(1, n_out, 509, device=dev), torch.arange(n_out - 128, n_out, device=dev)])
    q = buf.out_coords[rows, 1:].long()
    ref = torch.zeros((len(rows), C_out), dtype=torch.float64, device=dev)
    for k in range(27):
        p = 2 * q + torch.tensor([k // 9, k // 3 % 3, k % 3], device=dev)
        inside = (p < torch.tensor([X, Y, Z], device=dev)).all(dim=1)
        ref[inside] += feat[((p[:, 0] * Y + p[:, 1]) * Z + p[:, 2])[inside]].double() @ weight[k].double()
    got = buf.feat_out[rows].double()
    del buf, coords, feat
    torch.cuda.empty_cache()
    assert float((got - ref).abs().max() / ref.abs().max()) <= 1e-5


@pytest.mark.parametrize("K,C_in,C_out,n,dtype", [(3, 64, 64, 64 * 513, "f16"), (3, 64, 64, 64 * 2048 + 1, "bf16"), (3, 32, 64, 64 * 3072, "f16"), (3, 256, 256, 64 * 81, "f16"),
                                                  (5, 32, 32, 64 * 600 + 63, "bf16"), (3, 64, 64, 64 * 300 + 7, "f32"), (5, 32, 16, 64 * 1000 + 1, "f32"), (7, 32, 64, 64 * 520 + 5, "f16")])
def test_tiles_in_the_order_of_their_density(K, C_in, C_out, n, dtype):
    """First and last size of the rule, one window of 2,048 tiles and two, part-filled runs: every tile is computed whatever the map's
    bytes say, with the same bits, and as the oracle has it."""
    say(f"dense tiles first K={K} {C_in}->{C_out} {dtype} n={n}")
    import torch
    import oracle
    from paper_2402_07710_amd import binding as sc
    from tests.test_gpu_parity import rel_err, sampled_rows_reference
    tdt = {"f16": torch.float16, "bf16": torch.bfloat16, "f32": torch.float32}[dtype]
    scenes = [synth.lidar_scene(s) for s in range(-(-n // 50000))]
    for b, scene in enumerate(scenes):
        scene[:, 0] = b
    coords = np.ascontiguousarray(np.concatenate(scenes)[:n])
    feat, weight = synth.features(n, C_in, dtype, 3), synth.weights(K ** 3, C_in, C_out, dtype, 3)
    buf = sc.LayerBuffers(n, K, 1, "subm", C_in, C_out, dtype, "f32", device="cuda:0")
    c, f, w = torch.from_numpy(coords).to("cuda:0"), torch.from_numpy(feat).to("cuda:0").to(tdt), torch.from_numpy(weight).to("cuda:0").to(tdt)
    buf.layer(c, f, w)
    want = buf.feat_out.clone()
    tiles = -(-n // 64)
    density = buf.kmap[buf.kmap.numel() - -(-tiles // 256) * 256:][:tiles]            # the last part of the map
    masks = buf.kmap[256:256 + 16 * tiles * -(-K ** 3 // 32)].view(torch.int32).view(tiles, 4, -1).cpu().numpy().view(np.uint32)
    offsets = np.unpackbits(np.bitwise_or.reduce(masks, axis=1).view(np.uint8), axis=1).sum(axis=1).astype(int)
    assert np.array_equal(density.cpu().numpy(), offsets if K < 7 else offsets // 2)
    rng = np.random.default_rng(n)
    for fill in (rng.integers(0, 256, tiles), np.zeros(tiles), np.arange(tiles) % 4):
        density.copy_(torch.from_numpy(fill.astype(np.uint8)))
        buf.feat_out.fill_(float("nan"))
        buf.conv_fwd(f, w)
        assert torch.equal(buf.feat_out, want)
    rows = np.unique(np.concatenate([rng.choice(n, 1000, replace=False), np.arange(n - 70, n)]))
    err = rel_err(want.double().cpu().numpy()[rows], sampled_rows_reference(feat, weight, oracle.kmap(coords, K, 1, "subm"), rows)[rows])
    assert err <= 1e-5, err


@pytest.mark.parametrize("C_in,C_out,n", [(32, 64, 320 * 64), (32, 64, 320 * 64 + 1), (64, 64, 512 * 64 - 1), (64, 64, 512 * 64 + 1), (128, 128, 256 * 64), (128, 128, 256 * 64 + 1),
                                          (128, 32, 1000), (64, 80, 77), (128, 256, 64)])
def test_two_sets_of_wavefronts(C_in, C_out, n):
    """Both sides of the lines, two wavefronts across the rows (32 output channels), a part-filled block of output channels; tiles with
    odd and even numbers of offsets; the fused layer, which walks the same steps, gives the same bits."""
    say(f"two sets {C_in} -> {C_out}, n={n}")
    import torch
    from paper_2402_07710_amd import binding as sc
    from tests.test_gpu_parity import to_dev
    side = max(4, int(round((n * 8) ** (1 / 3))))
    coords = synth.uniform_cells(n, side, seed=C_in)
    coords = np.ascontiguousarray(coords[np.lexsort((coords[:, 3], coords[:, 2], coords[:, 1]))])
    check_layer(coords, 3, 1, "subm", C_in, C_out, "bf16", seed=n, out_dtype="f32", threads=16)
    check_layer(coords, 2, 2, "strided", C_in, C_out, "f16", seed=n, out_dtype="f32", threads=16)
    if C_out in (64, 128):
        c, f = torch.from_numpy(coords).to("cuda:0"), to_dev(synth.features(n, C_in, "f16", 1), "f16")
        w = to_dev(synth.weights(27, C_in, C_out, "f16", 1), "f16")
        outs = []
        for dims in (None, (1, side, side, side)):
            buf = sc.LayerBuffers(n, 3, 1, "subm", C_in, C_out, "f16", "f32", device="cuda:0", grid_dims=dims)
            buf.feat_out.fill_(float("nan"))
            (buf.layer if dims is None else buf.layer_fused)(c, f, w)
            outs.append(buf.feat_out)
        assert torch.equal(*outs)


@pytest.mark.parametrize("way,K,C_in,C_out", [("down", 2, 32, 32), ("down", 2, 32, 64), ("down", 2, 64, 64), ("up", 2, 64, 32), ("up", 2, 128, 64), ("up", 3, 32, 32),
                                              ("transposed", 2, 64, 32), ("transposed", 2, 64, 64)])
@pytest.mark.parametrize("n", [1, 64 * 8 + 1, 64 * 256 - 15, 64 * 256 + 1, 64 * 768 + 16, 64 * 1024 + 1, 64 * 1280 + 49, 64 * 2048 + 17])
def test_resident_kernels_deal_their_tiles(way, K, C_in, C_out, n):
    """Less than a tile per workgroup, one to four, and further rounds with fewer: one input per coarse cell, so that input and
    output rows are the same and a row is its input times the weights of its one offset."""
    say(f"resident kernel {way} K={K} {C_in}->{C_out} n={n}")
    import torch
    from paper_2402_07710_amd import binding as sc
    i, k = np.arange(n), np.arange(n) % K ** 3
    cells = np.stack([i % 50, i // 50 % 50, i // 2500], axis=1)
    xyz = cells * K + np.stack([k // (K * K), k // K % K, k % K], axis=1)
    coords = torch.from_numpy(np.concatenate([np.zeros((n, 1), dtype=np.int64), xyz], axis=1).astype(np.int32)).to("cuda:0")
    f = torch.from_numpy(synth.features(n, C_in, "f16", n)).to("cuda:0").half()
    w = torch.from_numpy(synth.weights(K ** 3, C_in, C_out, "f16", n)).to("cuda:0").half()
    want = torch.empty((n, C_out), dtype=torch.float64, device="cuda:0")
    for o in range(K ** 3):
        want[o::K ** 3] = f[o::K ** 3].double() @ w[o].double()
    down = sc.LayerBuffers(n, K, K, "strided", C_in, C_out, "f16", "f32", device="cuda:0")
    down.kmap_build(coords, standalone=True)
    outs = []
    if way == "down":
        for packed in (False, True):
            down.feat_out.fill_(float("nan"))
            (down.conv_fwd_packed if packed else down.conv_fwd)(f, sc.sc_conv_weight_pack(w, K) if packed else w)
            outs.append(down.feat_out[:n].clone())
    else:
        out = torch.full((n, C_out), float("nan"), dtype=torch.float32, device="cuda:0")
        if way == "up":
            sc.sc_conv_up_fwd(f, n, w, out, down.kmap, down.counts, K)
        else:
            inverse = torch.empty(sc.sc_kmap_bytes(n, K, K, "inverse"), dtype=torch.uint8, device="cuda:0")
            workspace = torch.empty(sc.sc_conv_workspace_bytes(K, C_in, C_out, "f16"), dtype=torch.uint8, device="cuda:0")
            sc.sc_kmap_transpose(down.kmap, n, K, K, down.counts, inverse)
            sc.sc_conv_fwd(f, w, out, inverse, down.counts, K, K, "inverse", workspace, n_map=n)
            outs.append(torch.full_like(out, float("nan")))
            sc.sc_conv_fwd_packed(f, sc.sc_conv_weight_pack(w, K), C_out, outs[0], inverse, down.counts, K, K, "inverse", n_map=n)
        outs.append(out)
    for got in outs:            # sums of up to 128 products in 32 bits
        assert float((got.double() - want).abs().max() / want.abs().max()) <= 1e-5


@pytest.mark.parametrize("n", [64 * 256, 64 * 256 + 1, 64 * 512, 64 * 512 + 1, 64 * 768 + 33, 64 * 1024, 64 * 1024 + 1])
def test_resident_3x3x3_kernel_deals_its_tiles(n):
    """Both numbers of tiles per workgroup at their ends, packed and raw weights and the fused form: the same bits, as the oracle has them."""
    say(f"resident kernel 3x3x3 n={n}")
    import torch
    import oracle
    from paper_2402_07710_amd import binding as sc
    from tests.test_gpu_parity import rel_err, sampled_rows_reference
    scenes = [synth.lidar_scene(s) for s in range(-(-n // 50000))]
    for b, scene in enumerate(scenes):
        scene[:, 0] = b
    coords = np.ascontiguousarray(np.concatenate(scenes)[:n])
    feat, weight = synth.features(n, 32, "bf16", 3), synth.weights(27, 32, 32, "bf16", 3)
    c, f, w = torch.from_numpy(coords).to("cuda:0"), torch.from_numpy(feat).to("cuda:0").bfloat16(), torch.from_numpy(weight).to("cuda:0").bfloat16()
    buf = sc.LayerBuffers(n, 3, 1, "subm", 32, 32, "bf16", "f32", device="cuda:0", grid_dims=(len(scenes), 1408, 1600, 41))
    outs = []
    for run in (lambda: buf.layer(c, f, w), lambda: buf.conv_fwd_packed(f, sc.sc_conv_weight_pack(w, 3)), lambda: buf.layer_fused(c, f, w)):
        buf.feat_out.fill_(float("nan"))
        run()
        outs.append(buf.feat_out.clone())
    assert torch.equal(outs[0], outs[1]) and torch.equal(outs[0], outs[2])
    rng = np.random.default_rng(n)
    rows = np.unique(np.concatenate([rng.choice(n, 1000, replace=False), np.arange(n - 70, n)]))
    err = rel_err(outs[0].double().cpu().numpy()[rows], sampled_rows_reference(feat, weight, oracle.kmap(coords, 3, 1, "subm"), rows)[rows])
    assert err <= 1e-5, err


@pytest.mark.parametrize("K,stride,C_in,C_out,n", [(5, 1, 32, 32, 512 * 64), (5, 1, 32, 32, 512 * 64 + 1), (5, 1, 64, 64, 512 * 64 - 1), (5, 1, 128, 128, 256 * 64 + 1), (5, 1, 128, 32, 77),
                                                   (5, 1, 64, 80, 1000), (7, 1, 32, 48, 300), (7, 1, 64, 32, 65), (4, 2, 32, 64, 3000), (4, 4, 64, 32, 3000), (5, 2, 128, 64, 1)])
@pytest.mark.parametrize("dtype", ["f16", "bf16"])
def test_two_sets_of_wavefronts_beyond_27_offsets(K, stride, C_in, C_out, n, dtype):
    """Both sides of the line; lists of one entry to all K^3, odd numbers of steps among them, two wavefronts across the rows, a part-filled block."""
    say(f"two sets K={K} s={stride} {C_in} -> {C_out}, n={n} {dtype}")
    side = max(4, int(round((n * (2 if n < 5000 else 8)) ** (1 / 3))))
    coords = synth.uniform_cells(n, side, seed=C_in)
    coords = np.ascontiguousarray(coords[np.lexsort((coords[:, 3], coords[:, 2], coords[:, 1]))])
    check_layer(coords, K, stride, "subm" if stride == 1 else "strided", C_in, C_out, dtype, seed=n, out_dtype="f32", threads=16)


@pytest.mark.parametrize("K,stride,C_in,C_out,n", [(3, 2, 64, 64, 64 * 600), (3, 1, 64, 64, 64 * 600), (5, 1, 32, 32, 64 * 600), (3, 2, 128, 128, 64 * 300), (2, 2, 64, 128, 64 * 300),
                                                   (5, 2, 32, 64, 64 * 600), (4, 2, 64, 64, 64 * 321), (3, 1, 64, 64, 64 * 300), (3, 1, 64, 64, 64 * 3073),
                                                   (3, 1, 32, 64, 64 * 3329), (3, 2, 32, 64, 64 * 1793), (3, 1, 128, 128, 64 * 5121), (2, 2, 128, 128, 64 * 5121)])
def test_capacity_of_the_output_leaves_the_bits_of_a_row(K, stride, C_in, C_out, n):
    """Layers on both sides of the line for two sets of wavefronts: the first rows alone, in a buffer small enough for the other
    side, are the whole layer's rows bit for bit, with raw and with packed weights.  A map too large to say how dense its tiles are; and the
    sizes from which the streaming kernel takes the whole layer and the general one its first rows."""
    say(f"capacity K={K} s={stride} {C_in}->{C_out} n={n}")
    import torch
    from paper_2402_07710_amd import binding as sc
    from tests.test_gpu_parity import to_dev
    mode = "subm" if stride == 1 else "strided"
    coords = torch.from_numpy(synth.uniform_cells(n, 50 if n < 100_000 else 80, seed=4)).to("cuda:0")
    feat, weight = to_dev(synth.features(n, C_in, "f16", 4), "f16"), to_dev(synth.weights(K ** 3, C_in, C_out, "f16", 4), "f16")
    buf = sc.LayerBuffers(n, K, stride, mode, C_in, C_out, "f16", "f32", device="cuda:0")
    buf.layer(coords, feat, weight)
    some = torch.full((64 * (100 if n < 100_000 else 900) + 5, C_out), float("nan"), dtype=torch.float32, device="cuda:0")
    assert int(buf.read_counts().n_out) >= len(some)
    sc.sc_conv_fwd(feat, weight, some, buf.kmap, buf.counts, K, stride, mode, buf.workspace)
    assert torch.equal(some, buf.feat_out[:len(some)])
    some.fill_(float("nan"))
    sc.sc_conv_fwd_packed(feat, sc.sc_conv_weight_pack(weight, K), C_out, some, buf.kmap, buf.counts, K, stride, mode)
    assert torch.equal(some, buf.feat_out[:len(some)])


@pytest.mark.parametrize("way,n", [("down", 64 * 256), ("down", 64 * 256 + 1), ("up", 64 * 192), ("up", 64 * 192 + 1), ("up", 64 * 224)])
def test_256_channels_with_one_and_two_output_blocks_per_wavefront(way, n):
    """Both sides of the lines for K == stride and for inverse maps: one input per coarse cell, so that a row is its input
    times the weights of its one offset."""
    say(f"256 -> 256 {way} n={n}")
    import torch
    from paper_2402_07710_amd import binding as sc
    i, k = np.arange(n), np.arange(n) % 8
    xyz = np.stack([i % 50, i // 50 % 50, i // 2500], axis=1) * 2 + np.stack([k // 4, k // 2 % 2, k % 2], axis=1)
    coords = torch.from_numpy(np.concatenate([np.zeros((n, 1), dtype=np.int64), xyz], axis=1).astype(np.int32)).to("cuda:0")
    f = torch.from_numpy(synth.features(n, 256, "f16", n)).to("cuda:0").half()
    w = torch.from_numpy(synth.weights(8, 256, 256, "f16", n)).to("cuda:0").half()
    want = torch.empty((n, 256), dtype=torch.float64, device="cuda:0")
    for o in range(8):
        want[o::8] = f[o::8].double() @ w[o].double()
    down = sc.LayerBuffers(n, 2, 2, "strided", 256, 256, "f16", "f32", device="cuda:0")
    down.kmap_build(coords, standalone=True)
    got = torch.full((n, 256), float("nan"), dtype=torch.float32, device="cuda:0")
    if way == "down":
        down.feat_out.fill_(float("nan"))
        down.conv_fwd(f, w)
        got = down.feat_out[:n]
    else:
        inverse = torch.empty(sc.sc_kmap_bytes(n, 2, 2, "inverse"), dtype=torch.uint8, device="cuda:0")
        sc.sc_kmap_transpose(down.kmap, n, 2, 2, down.counts, inverse)
        sc.sc_conv_fwd(f, w, got, inverse, down.counts, 2, 2, "inverse", down.workspace, n_map=n)
    assert float((got.double() - want).abs().max() / want.abs().max()) <= 1e-5            # sums of 256 products in 32 bits
