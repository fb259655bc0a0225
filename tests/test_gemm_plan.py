"""The plan of split products, on the host: what a product asks for as workspace over random shapes of every layout."""
import random


def test_workspace_of_a_product_is_bounded_and_made_of_whole_partial_sums():
    from paper_2602_05145_amd import binding as B
    rng = random.Random(11)
    split = 0
    for _ in range(4000):
        layout, out = rng.randrange(3), rng.randrange(2)
        m, n, k = (max(8, int(2 ** rng.uniform(3, 15)) // 8 * 8) for _ in range(3))
        if layout == 2:
            k += rng.randrange(8)                       # any number of rows
        elif rng.random() < 0.5:
            m += rng.randrange(8)
        need = B.tide_gemm_workspace_bytes(layout, m, n, k, out)
        big, small = -(-m // 256) * -(-n // 256), -(-m // 128) * -(-n // 128)
        assert 0 <= need <= 64 << 20                    # a partial sum of every CU, or of two blocks per CU
        assert need % (128 * 128 * 4) == 0
        if big >= 256 if out == 1 else 128 <= big < 200:
            assert need == 0
        if need:
            split += 1
            assert k > 4 * 64                           # a part keeps four slabs or more
            if big < 200:                               # every tile is split, into two parts or more
                parts = need // (128 * 128 * 4)
                assert parts % small == 0 and parts // small >= 2 or parts % (4 * big) == 0 and parts // (4 * big) >= 2
    assert split > 500
    assert B.tide_gemm_workspace_bytes(0, 0, 8, 8, 1) == 0 and B.tide_gemm_workspace_bytes(3, 8, 8, 8, 1) == 0
    assert B.tide_gemm_workspace_bytes(0, 128, 128, 8004, 1) == 0     # K-major rows that no 16-byte piece fits: not this kernel
