"""Which kernel a product of a worker step takes, at the borders of the rules (host only, no GPU call)."""
import pytest

import als_inputs as I
import paper_2401_09135_amd as A

F32, BF16 = A.ALS_DTYPE_F32, A.ALS_DTYPE_BF16
MIB = 1 << 20


@pytest.mark.parametrize("M,N,K,layout,epi,out,want", [
    (16384, 3584, 896, (0, 0), 2, BF16, "256x256/4 split 1"),      # whole rounds of 256 x 256 tiles
    (2560, 1024, 896, (0, 0), 0, BF16, "deep 128x128"),            # 160 tiles of 128 x 128, and one row of them less
    (2432, 1024, 896, (0, 0), 0, BF16, "deep 64x64"),
    (8192, 512, 512, (0, 0), 0, BF16, "256x256/4 split 1"),        # 64 tiles of 256 x 256, and two less
    (7936, 512, 512, (0, 0), 0, BF16, "deep 128x128"),
    (512, 512, 512, (0, 1), 0, F32, "any 32x32/8"),                # 16 of them, K from 512 on
    (512, 512, 448, (0, 1), 0, F32, "deep 64x64"),
    (600, 960, 320, (0, 0), 0, BF16, "any 64x64/2"),               # rows that are no multiple of a tile
    (600, 5003, 320, (0, 0), 0, BF16, "any 128x64/2"),
])
def test_bf16_products(M, N, K, layout, epi, out, want):
    assert A.gemm_route(M, N, K, *layout, BF16, out, epi) == want


@pytest.mark.parametrize("dtype", [F32, BF16])
def test_products_with_the_matrix_cores_off(dtype):
    for M in (600, 16384):
        for layout in ((0, 0), (0, 1), (1, 0)):
            assert A.gemm_route(M, 896, 896, *layout, dtype, flags=1) == "vector"
            assert A.gemm_route(M, 896, 896, *layout, dtype) != "vector"


@pytest.mark.parametrize("M,N,K,ws,want", [
    (1024, 128, 32000, 64 * MIB, "any 32x32/8"), (128, 256, 8192, 64 * MIB, "any 32x32/8"),   # no 256 x 256 tile to split
    (1024, 128, 32000, 0, "any 32x32/8"),                                                     # (nothing to do with a workspace)
    (8192, 128, 32000, 64 * MIB, "deep 64x64"),
    (1024, 256, 32000, 64 * MIB, "256x256/4 split 50"),
])
def test_input_gradient_of_the_output_matrix(M, N, K, ws, want):
    assert A.gemm_route(M, N, K, 0, 1, ws_bytes=ws) == want


@pytest.mark.parametrize("M,N,K,ws,want", [
    (2048, 1024, 1664, 64 * MIB, "any 128x64/2"), (640, 3584, 1984, 64 * MIB, "256x256/4 split 4"),   # one round of tiles that share K, two
    (384, 3072, 2048, 64 * MIB, "256x256/4 split 4"), (384, 3072, 2048, 0, "any 64x64/2"),
    (128, 2304, 1280, 64 * MIB, "any 32x32/8"), (128, 2304, 1920, 64 * MIB, "128x128/2 split 4"),
    (256, 512, 2048, 64 * MIB, "any 32x32/8"), (256, 512, 2112, 64 * MIB, "256x256/4 split 4"),
])
def test_weight_gradient_of_few_tiles(M, N, K, ws, want):
    assert A.gemm_route(M, N, K, 1, 0, ws_bytes=ws) == want


@pytest.mark.parametrize("dtype,want", [(BF16, "any 128x128"), (F32, "f32 128x128")])
def test_large_products_of_any_shape(dtype, want):
    """131072 tokens and an odd vocabulary: 4.2 and 6.4 million tiles of 32 x 32, which no kernel launches at that size."""
    for V in (33001, 50257):
        assert A.gemm_route(131072, V, 256, in_dtype=dtype, out_dtype=dtype) == want
        assert A.gemm_route(131072, 256, V, 0, 1, in_dtype=dtype) == want
    # the last grid that has fewer than 2^32 threads
    assert A.gemm_route(1 << 22, 512 * 128 - 1, 64, in_dtype=dtype, out_dtype=dtype) == "vector"
    assert A.gemm_route(1 << 22, 511 * 128 - 1, 64, in_dtype=dtype, out_dtype=dtype) == want


def test_gelu_with_fp32_outputs_has_vector_code_only():
    for M in (512, 500):
        assert A.gemm_route(M, 512, 512, out_dtype=F32, epi=2) == "vector"
        assert A.gemm_route(M, 512, 512, out_dtype=BF16, epi=2) != "vector"


@pytest.mark.parametrize("M,N,K,layout,want", [
    (256, 256, 256, (0, 0), "f32 32x32 natural"), (288, 256, 256, (0, 0), "f32 32x32 natural"),   # no border in the number of tiles
    (1024, 704, 256, (1, 0), "f32 32x32 natural"), (1024, 704, 257, (1, 0), "f32 32x32/4"),       # up to 191 tiles of 64 x 64
    (1024, 704, 511, (0, 1), "f32 32x32/4"), (1024, 704, 512, (0, 1), "f32 32x32/8"),
    (1024, 768, 256, (0, 1), "f32 64x64/2"), (2048, 2048, 256, (0, 1), "f32 128x128"),
])
def test_fp32_products(M, N, K, layout, want):
    assert A.gemm_route(M, N, K, *layout, F32) == want


@pytest.mark.parametrize("T,V,n,want", [
    (256, 256, 1, "counting"), (256, 256, 200, "counting"), (256, 256, 400, "sort in LDS"),
    (512, 1024, 50, "counting"), (512, 1024, 100, "sort in LDS"),        # 39 and 79 million comparisons: 6.7 us counted, 13; sorted 10
    (2048, 4096, 4, "counting"), (2048, 4096, 16, "sort in LDS"),        # 7.2 and 20.5 us; 12
    (1024, 32000, 4, "counting"), (1024, 32000, 8, "sort in LDS"),       # 15 and 27; 21
    (8192, 1024, 1, "counting"), (8192, 1024, 2, "sort in LDS"),         # 13 and 21; 18
    (1024, 50257, 2, "counting"), (1024, 50257, 4, "sort"),              # past 150 million comparisons
    (12288, 2, 1, "sort in LDS"), (16384, 32000, 1, "sort in LDS"), (16385, 100, 1, "sort"), (512, 131073, 1, "sort"),
])
def test_order_of_a_calls_tokens(T, V, n, want):
    """Counting takes longer with every step of a call, the sort takes the steps side by side."""
    assert A.token_order_route(T, V, n) == want


@pytest.mark.parametrize("T,V,d,want", [
    (512, 8192, 256, "one launch"), (513, 8192, 256, "two launches"), (512, 8193, 256, "two launches"),
    (512, 256, 512, "one launch"), (512, 256, 576, "two launches"), (384, 255, 512, "one launch"), (385, 255, 512, "two launches"),
    (256, 8192, 1024, "one launch"), (257, 8192, 1024, "two launches"), (512, 8192, 1024, "two launches"),  # 32 us in one launch, 18 in two
    (32, 64, 64, "one launch"),
])
def test_embedding_gradient(T, V, d, want):
    """One launch leaves the longest list to one workgroup, once for every 256 columns."""
    assert A.embed_grad_route(T, V, d) == want


def _config(name, workers, **kw):
    cfg = A.Config.from_workload(dict(I.workload(name), **kw))
    cfg.n_workers = workers
    return cfg


@pytest.mark.parametrize("name,kw", [("tiny", {}), ("mini_bf16", {}), ("mini_bf16", dict(B=16, V=8192)), ("mini_bf16", dict(B=32, V=8192)),
                                     ("mini_bf16", dict(d=512, h=8, ff=2048, B=16)), ("lm20m", {}), ("lm150m_b1", {})])
def test_steps_replayed_as_graphs(name, kw):
    """Four hardware queues: workers on more streams do not run side by side, so more of them replay nothing that four do not."""
    four = A.replay_route(_config(name, 4, **kw), 4)
    assert four == (name == "tiny" or kw in ({}, dict(B=16, V=8192)) and name == "mini_bf16")
    for streams in (8, 16, 64):
        assert A.replay_route(_config(name, 64, **kw), streams) == four
    for workers, streams in ((1, 1), (2, 2), (4, 2), (64, 1), (2, 16)):       # the chip is the slower side
        assert not A.replay_route(_config(name, workers, **kw), streams)
