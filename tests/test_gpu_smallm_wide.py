"""The product for 33 to 64 tokens (k_smallm_wide) at the edges of its tiles, K-steps and token groups, against the oracle;
the bits are those of the kernel for up to 32 tokens, and batches under one X and under tokens of their own give the bits of
the single product."""
import numpy as np
import pytest

from oracle import egt_oracle as O
from paper_2605_11582_amd import binding as B, synth
import gpu_common as G

pytestmark = pytest.mark.gpu


def _case(rows, cols, g, seed):
    w = synth.weights(rows, cols, seed)
    mask = O.prune_n4_magnitude(w, 2)
    return B.pack_2bitcsr(w, mask, 2, g, B.VAL_INT4), O.pack_2bitcsr(w, mask, 2, g, O.VAL_INT4)


# rows: part of a tile, one, 2 to 4 and 5 tiles a workgroup; cols: part of a K-step, 1 to 8 waves, 1 to 4 phases with an odd and
# an even last one, the last of them in some waves only; tokens: the ends of both token-group counts
@pytest.mark.parametrize("rows,cols,g,M", [
    (1, 64, 64, 33), (17, 192, 64, 48), (40, 512, 128, 49), (33, 2048, 128, 64), (35, 2112, 64, 33), (50, 4096, 256, 64),
    (31, 4160, 64, 47), (64, 6208, 64, 63), (20, 8192, 512, 34),
    (4100, 256, 128, 40), (8200, 320, 64, 57), (12300, 64, 64, 48), (12300, 128, 128, 64), (16400, 192, 64, 35), (16400, 64, 64, 64)])
def test_products_for_many_tokens(rows, cols, g, M):
    print(f"case smallm wide {rows}x{cols} g={g} M={M}", flush=True)
    p, o = _case(rows, cols, g, 7000 + M + cols)
    X = synth.activation_rows(M, cols, 7100 + M)
    Y_ref, A_ref = O.gemm_smallm(o, X)
    for pad in (0, 6, 7):        # 8-byte stores of four rows, the 2-byte fallback, odd strides
        Y = G.run_sparse_gemm(p, X, ldx_pad=pad - pad % 2, ldy_pad=pad)
        G.assert_close(Y, Y_ref, A_ref, f"smallm wide {rows}x{cols} M={M} pad={pad}")


# rows of more than 2048 columns: 32 tokens go to k_sparse_smallm_ks there (test_kernel_routes), which splits K over as many waves
MORE_THAN_2048 = [(1, 2112, 64, 33), (50, 4160, 64, 64), (31, 11008, 128, 47), (4100, 2304, 128, 48), (8203, 2176, 64, 57),
                  (12300, 2112, 64, 49), (16400, 2560, 512, 64)]


@pytest.mark.parametrize("rows,cols,g,M", MORE_THAN_2048)
def test_the_bits_are_those_of_the_kernel_for_fewer_tokens(rows, cols, g, M):
    print(f"case smallm wide bits {rows}x{cols} g={g} M={M}", flush=True)
    w = synth.weights(rows, cols, 7500 + cols)
    p = B.pack_2bitcsr(w, B.prune_n4(w, 2), 2, g, B.VAL_INT4)
    X = synth.activation_rows(M, cols, 7501)
    Y = G.run_sparse_gemm(p, X).view(np.uint16)
    for k in (0, M - 32):                             # the first 32 tokens and the last: every token, other token groups
        assert np.array_equal(Y[k:k + 32], G.run_sparse_gemm(p, X[k:k + 32]).view(np.uint16)), k


@pytest.mark.parametrize("rows,cols,M,count", [(4234, 1792, 50, 3), (2064, 4096, 33, 4), (300, 640, 64, 2), (4500, 2112, 40, 2)])
@pytest.mark.parametrize("shared", [True, False])
def test_batches_for_many_tokens_give_the_bits_of_the_single_product(rows, cols, M, count, shared):
    torch = G.torch_mod()
    print(f"case smallm wide batch {rows}x{cols} M={M} count={count} shared={shared}", flush=True)
    packed = [_case(rows, cols, 64, 7200 + k)[0].to("cuda") for k in range(count)]
    xs = [G.to_dev(synth.activation_rows(M, cols, 7300 + (0 if shared else k)).view(np.uint16)).view(torch.float16) for k in range(count)]
    if shared:
        xs = [xs[0]] * count
    one = [torch.zeros((M, rows), dtype=torch.float16, device="cuda") for _ in range(count)]
    many = [torch.full((M, rows), 7, dtype=torch.float16, device="cuda") for _ in range(count)]
    for w, x, y in zip(packed, xs, one):
        B.sparse_gemm_smallm(w, x, y)
    B.sparse_gemm_smallm_batch(packed, xs, many)
    torch.cuda.synchronize()
    for a, b in zip(one, many):
        assert torch.equal(a, b)


def test_a_broken_row_pointer_marks_its_row_only():
    torch = G.torch_mod()
    print("case smallm wide broken row pointer", flush=True)
    p = _case(4500, 512, 128, 7400)[0]
    X = G.to_dev(synth.activation_rows(40, 512, 7401).view(np.uint16)).view(torch.float16)
    good = torch.zeros((40, 4500), dtype=torch.float16, device="cuda")
    B.sparse_gemm_smallm(p.to("cuda"), X, good)
    p.row_ptr[4300] += 8
    Y = torch.zeros_like(good)
    B.sparse_gemm_smallm(p.to("cuda"), X, Y)
    torch.cuda.synchronize()
    assert torch.isnan(Y[:, 4300]).all()
    Y[:, 4300] = good[:, 4300]
    assert torch.equal(Y, good)
