"""The block forms of plans with 64x64 tiles, on the GPU.

The GEMM of such a plan computes 128x128, 64x64, 64x32 or 32x32 outputs per
workgroup, chosen by the number of tiles against the plan's wave width (parts
of a tile only without counters). Every form must give the same bits, at the
edges of the rule, with an odd number of tile rows and columns (128x128 blocks
that reach past the output) and every remainder of the k steps.
"""
import numpy as np
import pytest

import oracle
import paper_2504_19519_amd as fo
import workloads
from gpu_util import assert_close_bits, dev_plan, empty16, from_dev, say, to_dev, torch_mod, zeros_u32

pytestmark = pytest.mark.gpu

M, N = 192, 320          # 15 tiles
# W = modelled compute units: 15 tiles <= W/4, > W/4, <= W/2, > W/2, <= 2 W, > 2 W
WIDTHS = [60, 59, 30, 29, 8, 7]


@pytest.mark.parametrize("dtype", ["fp16", "bf16"])
@pytest.mark.parametrize("K", [64, 128, 192, 448, 640])
def test_block_forms(dtype, K):
    torch = torch_mod()
    say(f"[gemm blocks] {M}x{N}x{K} {dtype}")
    rng = np.random.default_rng(K)
    A = workloads.to_bits(rng.uniform(-1, 1, (M, K)), dtype)
    W = workloads.to_bits(rng.uniform(-1, 1, (N, K)) / np.sqrt(K), dtype)
    dA, dW = to_dev(A), to_dev(W)
    plain = None
    for cus in WIDTHS:
        for pattern, nd in [("rowmajor", 0), ("tile", 0), ("subtile", 4), ("subtoken", 3)]:
            sigma = rng.permutation(nd) if pattern == "subtile" else None
            bucket = rng.integers(0, nd, M) if pattern == "subtoken" else None
            T = -(-15 // cus)
            sizes = [1] * T
            plan = fo.plan_groups(M, N, K, dtype=dtype, tile_m=64, tile_n=64, num_cus=cus, pattern=pattern,
                                  num_dest=nd, dest_perm=sigma, row_bucket=bucket, sizes=sizes)
            o = oracle.make_plan(M, N, 64, 64, num_cus=cus, order="xcd", group_m=4, num_xcds=8, pattern=pattern,
                                 num_dest=nd, sigma=sigma, bucket=bucket, sizes=sizes, unit="waves")
            dp = dev_plan(plan)
            for counters in (None, zeros_u32(plan.num_counters)):
                C = empty16(M * N, dtype)
                fo.gemm_signal_reorder(plan, dp, dA, dW, C, counters)
                torch.cuda.synchronize()
                got = from_dev(C)[:M * N]
                if plain is None:
                    plain = got
                    assert_close_bits(got, oracle.gemm_ref(A, W, dtype).reshape(-1), dtype, "GEMM")
                what = f"W={cus} {pattern} {'signalled' if counters is not None else 'unsignalled'}"
                np.testing.assert_array_equal(got, plain[oracle.reorder_index(o)], err_msg=what)
                if counters is not None:
                    c = counters.cpu().numpy()
                    np.testing.assert_array_equal(c[:plan.P], np.array(o.targets), err_msg=what)
                    np.testing.assert_array_equal(c[plan.P:plan.P + fo.DISPENSER_WORDS], 0, err_msg=what)


@pytest.mark.parametrize("reserved", [0, 3])        # (with reserved units, blocks run one to a unit)
@pytest.mark.parametrize("tile_n,widths", [(128, [12, 11, 5, 4]), (256, [24, 12, 11, 5, 4])])
@pytest.mark.parametrize("dtype,K", [("fp16", 64), ("bf16", 192), ("fp16", 448)])
def test_parts_of_larger_tiles(tile_n, widths, dtype, K, reserved):
    # 6 tiles of 256 x tile_n: unsignalled launches take 128x128 blocks where
    # the last wave is emptier in whole tiles (at most W / 2, and just past W),
    # signalled ones whole tiles; the bits are the same
    torch = torch_mod()
    M, N = 512, 3 * tile_n
    say(f"[gemm parts] {M}x{N}x{K} tile 256x{tile_n} {dtype}")
    rng = np.random.default_rng(K)
    A = workloads.to_bits(rng.uniform(-1, 1, (M, K)), dtype)
    W = workloads.to_bits(rng.uniform(-1, 1, (N, K)) / np.sqrt(K), dtype)
    dA, dW = to_dev(A), to_dev(W)
    plain = None
    for cus in widths:
        for pattern, nd in [("rowmajor", 0), ("tile", 0), ("subtile", 4), ("subtoken", 3)]:
            sigma = rng.permutation(nd) if pattern == "subtile" else None
            bucket = rng.integers(0, nd, M) if pattern == "subtoken" else None
            sizes = [1] * -(-6 // cus)
            plan = fo.plan_groups(M, N, K, dtype=dtype, tile_m=256, tile_n=tile_n, num_cus=cus + reserved,
                                  reserved_cus=reserved, pattern=pattern,
                                  num_dest=nd, dest_perm=sigma, row_bucket=bucket, sizes=sizes)
            o = oracle.make_plan(M, N, 256, tile_n, num_cus=cus + reserved, reserved_cus=reserved, order="xcd",
                                 group_m=4, num_xcds=8, pattern=pattern,
                                 num_dest=nd, sigma=sigma, bucket=bucket, sizes=sizes, unit="waves")
            dp = dev_plan(plan)
            for counters in (None, zeros_u32(plan.num_counters)):
                C = empty16(M * N, dtype)
                fo.gemm_signal_reorder(plan, dp, dA, dW, C, counters)
                torch.cuda.synchronize()
                got = from_dev(C)[:M * N]
                if plain is None:
                    plain = got
                    assert_close_bits(got, oracle.gemm_ref(A, W, dtype).reshape(-1), dtype, "GEMM")
                np.testing.assert_array_equal(got, plain[oracle.reorder_index(o)],
                                              err_msg=f"W={cus} {pattern} {'signalled' if counters is not None else ''}")


@pytest.mark.parametrize("order", ["grouped", "xcd"])
@pytest.mark.parametrize("tile,grid", [((64, 64), (4, 4)), ((64, 64), (4, 1)), ((64, 64), (4, 2)),
                                       ((256, 128), (2, 3)), ((256, 256), (2, 1))])
def test_bands_taller_than_the_output(tile, grid, order):
    # "one band over everything" written as a large number (powers of two whose
    # double, or whose product with the columns of a block grid, leaves 32 bits):
    # the bits of any other order
    torch = torch_mod()
    K, (M, N) = 128, (tile[0] * grid[0], tile[1] * grid[1])
    tiles = grid[0] * grid[1]
    say(f"[gemm tall bands] {M}x{N}x{K} tile {tile} {order}")
    rng = np.random.default_rng(tiles)
    A = workloads.to_bits(rng.uniform(-1, 1, (M, K)), "bf16")
    W = workloads.to_bits(rng.uniform(-1, 1, (N, K)) / np.sqrt(K), "bf16")
    dA, dW = to_dev(A), to_dev(W)
    plain = None
    for group_m, xcds in [(1, 8), (1 << 28, 8), (1 << 29, 3), (1 << 30, 8), ((1 << 31) - 1, 8), (4, (1 << 31) - 20)]:
        for cus in (4 * tiles, 2 * tiles, tiles, 2):      # 32x32, 64x32, whole tiles, 128x128 blocks
            kw = dict(num_cus=cus, order=order, group_m=group_m, num_xcds=xcds, pattern="tile",
                      sizes=[-(-tiles // cus)])
            plan = fo.plan_groups(M, N, K, dtype="bf16", tile_m=tile[0], tile_n=tile[1], **kw)
            o = oracle.make_plan(M, N, *tile, unit="waves", **kw)
            dp = dev_plan(plan)
            for counters in (None, zeros_u32(plan.num_counters)):
                C = empty16(M * N, "bf16")
                fo.gemm_signal_reorder(plan, dp, dA, dW, C, counters)
                torch.cuda.synchronize()
                got = from_dev(C)[:M * N]
                if plain is None:
                    plain = np.empty_like(got)
                    plain[oracle.reorder_index(o)] = got
                    assert_close_bits(plain, oracle.gemm_ref(A, W, "bf16").reshape(-1), "bf16", "GEMM")
                np.testing.assert_array_equal(got, plain[oracle.reorder_index(o)], err_msg=f"{group_m} {xcds} {cus}")


# tile rows and columns, compute units, reserved ones, order, band height, chiplets: 128x128 blocks (100 of them, and
# grids that reach past the output) over few workgroups, and 64x64 blocks (tiles in (W, 2 W]) that the reserved units
# keep from running in pairs
ROUNDS = [(20, 20, 5, 0, "xcd", 4, 8), (19, 21, 12, 0, "grouped", 3, 1), (19, 21, 7, 0, "xcd", 5, 3),
          (6, 9, 33, 3, "xcd", 4, 8), (7, 7, 27, 2, "grouped", 2, 1)]


@pytest.mark.parametrize("rows,cols,cus,reserved,order,band,xcds", ROUNDS)
@pytest.mark.parametrize("K", [64, 128, 192, 320])
def test_signalled_blocks_in_rounds(rows, cols, cus, reserved, order, band, xcds, K):
    # more blocks than workgroups: positions drawn from the position words, a
    # block's counts sent during the next one's first steps (or, when the loop is
    # shorter than the ring, ahead of it), the next block's loads ahead of the
    # stores. Every producer mode, launches in a row that clear the group
    # counters only, and runs with live consumers on a NaN-filled buffer: a count
    # that is sent before its tile is stored lets one read the NaNs in C.
    torch = torch_mod()
    M, N, dtype = 64 * rows, 64 * cols, "fp16"
    tiles, W = rows * cols, cus - reserved
    blocks = (rows + 1) // 2 * ((cols + 1) // 2) if tiles > 2 * W else tiles
    assert blocks > (2 * W if not reserved else W), "one block per workgroup"
    say(f"[signalled blocks] {M}x{N}x{K} W={W} {order} {band} {xcds}")
    rng = np.random.default_rng(K + tiles)
    A = workloads.to_bits(rng.uniform(-1, 1, (M, K)), dtype)
    Wt = workloads.to_bits(rng.uniform(-1, 1, (N, K)) / np.sqrt(K), dtype)
    dA, dW = to_dev(A), to_dev(Wt)
    peer = workloads.uniform_bits(M * N, 7, dtype)
    dP = to_dev(peer)
    s1, s2 = torch.cuda.Stream(), torch.cuda.Stream()
    plain_plan = fo.plan_groups(M, N, K, dtype=dtype, tile_m=64, tile_n=64, pattern="rowmajor", sizes=[-(-tiles // 256)])
    C = empty16(M * N, dtype)
    fo.gemm_signal_reorder(plain_plan, None, dA, dW, C, None)
    torch.cuda.synchronize()
    plain = from_dev(C)[:M * N]
    assert_close_bits(plain, oracle.gemm_ref(A, Wt, dtype).reshape(-1), dtype, "GEMM")
    T = -(-tiles // W)
    sizes = [1, T - 1] if T < 3 else [1, T // 2, T - 1 - T // 2]
    for pattern, nd in [("tile", 0), ("subtile", 4), ("subtoken", 3)]:
        kw = dict(num_cus=cus, reserved_cus=reserved, order=order, group_m=band, num_xcds=xcds, pattern=pattern,
                  num_dest=nd, sizes=sizes)
        sigma = rng.permutation(nd) if pattern == "subtile" else None
        bucket = rng.integers(0, nd, M) if pattern == "subtoken" else None
        plan = fo.plan_groups(M, N, K, dtype=dtype, tile_m=64, tile_n=64, dest_perm=sigma, row_bucket=bucket, **kw)
        o = oracle.make_plan(M, N, 64, 64, sigma=sigma, bucket=bucket, unit="waves", **kw)
        assert plan.P > 1
        dp, want = dev_plan(plan), plain[oracle.reorder_index(o)]
        sums = oracle.apply_consumer(o, want, peer if pattern != "subtoken" else None, dtype)
        C = empty16(M * N, dtype)                 # the unsignalled kernel's loop over blocks
        torch.cuda.synchronize()
        fo.gemm_signal_reorder(plan, dp, dA, dW, C, None)
        torch.cuda.synchronize()
        np.testing.assert_array_equal(from_dev(C)[:M * N], want, err_msg=f"{pattern} unsignalled")
        for mode in (0, 1, 2):
            ctr = zeros_u32(plan.num_counters)
            for launch in range(3):
                what = f"{pattern} mode {mode} launch {launch}"
                C = empty16(M * N, dtype)
                ctr[:plan.P].zero_()
                torch.cuda.synchronize()
                fo.gemm_signal_reorder(plan, dp, dA, dW, C, ctr, opts={"sync_producer": mode})
                torch.cuda.synchronize()
                np.testing.assert_array_equal(from_dev(C)[:M * N], want, err_msg=what)
                c = ctr.cpu().numpy()
                np.testing.assert_array_equal(c[:plan.P], np.array(o.targets), err_msg=what)
                np.testing.assert_array_equal(c[plan.P:plan.P + fo.DISPENSER_WORDS], 0, err_msg=what)
            C, dst, out, status = empty16(M * N, dtype), empty16(M * N, dtype), empty16(M * N, dtype), zeros_u32(1)
            torch.cuda.synchronize()
            fo.run_overlapped(plan, dp, dA, dW, C, dP if pattern != "subtoken" else None, dst, out, counters=ctr,
                              status_word=status, gemm_stream=s1, comm_stream=s2,
                              opts={"sync_producer": mode, "sync_consumer": mode, "consumer_blocks": 255})
            torch.cuda.synchronize()
            what = f"{pattern} mode {mode} with consumers"
            assert int(status.cpu()[0]) == 0, what
            np.testing.assert_array_equal(from_dev(C)[:M * N], want, err_msg=what)
            np.testing.assert_array_equal(from_dev(dst)[:M * N], sums, err_msg=what)
            np.testing.assert_array_equal(from_dev(out)[:M * N], sums[oracle.post_index(o)], err_msg=what)
