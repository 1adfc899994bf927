"""Weight gradients within the rounding errors of their own sums: a lost chunk of rows, or one row of another
window, is outside the bound (which the tests without a GPU check)."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

U32 = 2.0 ** -24
STEP = 16          # rows that one step of a sum takes, in any order


def chunk_rows(M, T, tiles, blocks=512):
    """Rows per chunk of a product with `tiles` output tiles of 128 x 128: whole windows, halved (down to 128
    rows) until `blocks` blocks have work."""
    rows = T
    while (M // rows) * tiles < blocks and rows % 256 == 0:
        rows //= 2
    return rows


def chunk_rows_256(M, T):
    """Rows per chunk of the 256 x 256 tile (0 where the 128 x 128 tiles are taken)."""
    rows = chunk_rows(M, T, 1, 192)
    return rows if rows >= 1024 and M // rows >= 192 else 0


def reduction_depth(chunks):
    """Additions of the chunks' sums: 16 groups in order and then the groups from 128 chunks on."""
    return -(-chunks // 16) + 16 if chunks >= 128 else chunks


def product_bound(A, B, rows):
    """A^T B [K, N] of float64 A [M, K], B [M, N], and a bound on the error of fp32 sums of exact (or fused)
    products over chunks of `rows` rows, STEP rows at a time: each of a step's STEP additions errs by at
    most 2 u times the magnitude of what it adds to, and that is at most |sum before the step| + the step's
    sum of |products| (2 u, not u: the matrix instruction may truncate); then the chunks are added."""
    ref = torch.zeros((A.shape[1], B.shape[1]), dtype=torch.float64, device=A.device)
    bound, parts = torch.zeros_like(ref), torch.zeros_like(ref)
    n = A.shape[0] // rows
    for c in range(n):
        a = A[c * rows:(c + 1) * rows].reshape(rows // STEP, STEP, -1).transpose(1, 2).contiguous()
        b = B[c * rows:(c + 1) * rows].reshape(rows // STEP, STEP, -1).contiguous()
        p = torch.bmm(a, b)
        s = torch.cumsum(p, 0)
        bound += STEP * 2 * U32 * ((s - p).abs().sum(0) + torch.bmm(a.abs(), b.abs()).sum(0))
        ref += s[-1]
        parts += s[-1].abs()
    return ref, 1.01 * (bound + reduction_depth(n) * U32 * parts)


def column_bound(A, rows):
    """Column sums of A and their bound: eight threads add every eighth run of rows, then each other."""
    s = A.reshape(-1, rows, A.shape[1])
    parts, n = s.sum(1), s.shape[0]
    return A.sum(0), 1.01 * U32 * ((rows // 8 + 8) * A.abs().sum(0) + reduction_depth(n) * parts.abs().sum(0))


def check(label, got, ref, bound):
    err = (got - ref).abs()
    print(f"{label}: max error / bound = {float((err / (bound + 1e-300)).max()):.3g}", flush=True)
    assert bool((err <= bound).all()), label


# ---------------------------------------------------------------- the bound itself, on the CPU
@pytest.mark.parametrize("B,T,rows", [(192, 1024, 1024), (97, 2048, 1024), (201, 1152, 1152)])
def test_bound_rejects_lost_and_foreign_rows(B, T, rows):
    """fp32 sums in the kernels' chunks meet the bound; against references with a fault planted they do not:
    one chunk left out (nine of ten entries outside), one row of one window paired with the row before its
    window, one chunk left out of the column sums."""
    M, K, N = B * T, 16, 16
    rng = np.random.default_rng(B)
    A = rng.standard_normal((M, K)).astype(np.float32).astype(np.float64)
    X = rng.standard_normal((M, N)).astype(np.float32).astype(np.float64)
    got, sums = np.zeros((K, N), dtype=np.float32), np.zeros(K, dtype=np.float32)
    for c in range(M // rows):
        part, col = np.zeros((K, N), dtype=np.float32), np.zeros(K, dtype=np.float32)
        for a, x in zip(A[c * rows:(c + 1) * rows], X[c * rows:(c + 1) * rows]):
            part = (part + a[:, None] * x[None, :]).astype(np.float32)   # (one rounding, as a fused multiply-add)
            col = (col + a).astype(np.float32)
        got, sums = got + part, sums + col
    At, Xt = torch.from_numpy(A), torch.from_numpy(X)
    ref, bound = product_bound(At, Xt, rows)
    g = torch.from_numpy(got.astype(np.float64))
    check("product", g, ref, bound)
    c = 5
    lost = ref - At[c * rows:(c + 1) * rows].T @ Xt[c * rows:(c + 1) * rows]
    assert ((g - lost).abs() > bound).double().mean() > 0.9
    w = 7 * T
    foreign = ref + At[w][:, None] * Xt[w - 1][None, :]
    assert bool(((g - foreign).abs() > bound).any())
    cref, cbound = column_bound(At, rows)
    gs = torch.from_numpy(sums.astype(np.float64))
    # (added in order here: a depth of `rows`, eight times the kernels')
    check("columns", gs, cref, 8 * cbound)
    assert bool(((gs - (cref - At[c * rows:(c + 1) * rows].sum(0))).abs() > cbound).any())


# ---------------------------------------------------------------- the kernels
@pytest.mark.gpu
@pytest.mark.parametrize("prec,B,T,layer", [("bf16", 192, 1024, 9), ("bf16", 97, 2048, 28), ("bf16", 201, 1152, 5), ("bf16", 65, 1024, 19),
                                            ("bf16", 513, 128, 3), ("fp32", 65, 1024, 9), ("fp32", 513, 128, 3), ("fp32", 5, 640, 28)])
def test_weight_gradients_of_one_layer(prec, B, T, layer):
    """One layer's weight and bias gradients in float64 from the operands its kernels read."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from oracle.arch import FULL, layout
    from paper_2201_11133_amd import gwd, synth
    print(f"case: {prec} layer {layer}, B = {B}, T = {T}", flush=True)
    C, M = 128, B * T
    gen = torch.Generator(device="cuda").manual_seed(B + T)
    bufs = {k: torch.empty((M, 2 * C if k in ("pre", "dpre") else C), device="cuda")
            for k in ("x_in", "pre", "dskip", "dx_in", "dg", "g", "dpre", "dx_out")}
    u = torch.randn((B, T, 2), generator=gen, device="cuda")
    dz = torch.randn((B, T), generator=gen, device="cuda")
    m = gwd.Model(gwd.full_arch(), synth.full_weights(4), prec)
    m.capture_backward(layer, bufs)
    z, grad = torch.empty((B, T), device="cuda"), torch.empty(m.n_params, device="cuda")
    saved = torch.empty(gwd.lib.gwd_saved_bytes(m.h, B, T), dtype=torch.uint8, device="cuda")
    st = gwd._stream_handle(None)
    gwd.check(gwd.lib.gwd_forward_train(m.h, 0, u.data_ptr(), B, T, z.data_ptr(), saved.data_ptr(), st))
    gwd.check(gwd.lib.gwd_backward(m.h, 0, u.data_ptr(), B, T, saved.data_ptr(), dz.data_ptr(), grad.data_ptr(), None, st))
    torch.cuda.synchronize()
    m.capture_backward(-1)
    m.close()
    grads, o = {}, 0
    for name, shape, _ in layout(FULL):
        n = int(np.prod(shape))
        grads[name] = grad[o:o + n].double().reshape(shape)
        o += n
    op = (lambda v: v.bfloat16().double()) if prec == "bf16" else (lambda v: v.double())   # as the products read them
    last = layer == FULL.n_layers - 1
    x, g, dpre = bufs["x_in"].double(), bufs["g"].double(), bufs["dpre"].double()
    # skip and residual in one product, 128 columns of g
    rows = chunk_rows(M, T, 1 if last else 2)
    check("d skip.W", grads[f"skip{layer}.W"], *product_bound(op(bufs["dskip"]), g, rows))
    if not last:
        check("d res.W", grads[f"res{layer}.W"], *product_bound(op(bufs["dx_in"]), g, rows))
        check("d res.b", grads[f"res{layer}.b"], *column_bound(bufs["dx_in"].double(), rows))
    # both taps in one product
    rows = (chunk_rows_256(M, T) if prec == "bf16" else 0) or chunk_rows(M, T, 4)
    d = FULL.dilation(layer)
    xd = torch.zeros((B, T, C), dtype=torch.float64, device="cuda")
    if d < T:
        xd[:, d:] = x.reshape(B, T, C)[:, :-d]
    check("d dil.W tap 1", grads[f"dil{layer}.W"][:, :, 1], *product_bound(dpre, x, rows))
    check("d dil.W tap 0", grads[f"dil{layer}.W"][:, :, 0], *product_bound(dpre, xd.reshape(M, C), rows))
    check("d dil.b", grads[f"dil{layer}.b"], *column_bound(dpre, rows))
