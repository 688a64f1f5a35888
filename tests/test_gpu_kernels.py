"""GPU parity of the single kernels, through the C ABI, against the CPU oracle on the same
seeded inputs: rotation and sparse projection within 2e-3 relative L2, Top-K indices equal."""
import numpy as np
import pytest
import torch

from oracle import larosa_oracle as O
from paper_2507_01299_amd import synth
from tests.gpu_util import REL_L2_TOL, rel_l2, stored_close, to_bits, to_dev

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def api(gpu_device):
    from paper_2507_01299_amd import api as A
    A.lib()
    return A


@pytest.fixture(scope="module")
def ws(api):
    return api.workspace(8, 32768, 32768, 32768)


def _heavy_vector(rng, B, d, dtype):
    v = rng.standard_normal((B, d)) * (np.arange(1, d + 1) ** -0.6)[None, :]
    v[:, rng.choice(d, 4, replace=False)] *= 20
    bits = O.encode16(v, dtype)
    return bits, O.decode16(bits, dtype)


@pytest.mark.parametrize("dtype", ["f16", "bf16"])
@pytest.mark.parametrize("B,d", [(1, 512), (3, 1096), (1, 8), (2, 2048)])
def test_rotate_matches_oracle(api, ws, dtype, B, d):
    print(f"rotate dtype={dtype} B={B} d={d}", flush=True)
    rng = np.random.default_rng(100 + d + B)
    Q = synth.planted_basis(d, seed=d)
    qb = O.encode16(Q, dtype)
    xb, x = _heavy_vector(rng, B, d, dtype)
    h = torch.zeros(B, d, dtype=api.torch_dtype(dtype), device="cuda:0")
    api.rotate(to_dev(xb, dtype), to_dev(qb, dtype), h, dtype, ws)
    torch.cuda.synchronize()
    want = O.round16(O.rotate(x, O.decode16(qb, dtype)), dtype)      # the output is a stored 16-bit tensor
    for b in range(B):
        stored_close(to_bits(h)[b], want[b], dtype, "rotate")
    # identity rotation returns the input bits
    eye = O.encode16(np.eye(d), dtype)
    api.rotate(to_dev(xb, dtype), to_dev(eye, dtype), h, dtype, ws)
    torch.cuda.synchronize()
    assert np.array_equal(to_bits(h), xb)


@pytest.mark.parametrize("dtype", ["f16", "bf16"])
@pytest.mark.parametrize("B,d,K", [(1, 512, 256), (1, 4096, 2457), (2, 4096, 1), (1, 4096, 4096), (3, 11008, 6604),
                                   (1, 14336, 8601), (2, 28672, 17203), (1, 32768, 5), (1, 8, 3), (4, 1000, 999),
                                   (1, 8192, 4915)])
def test_topk_indices_are_exact(api, dtype, B, d, K):
    print(f"topk dtype={dtype} B={B} d={d} K={K}", flush=True)
    rng = np.random.default_rng(7 * d + K)
    hb, _ = _heavy_vector(rng, B, d, dtype)
    idx = torch.full((B, K), -1, dtype=torch.int32, device="cuda:0")
    vals = torch.zeros(B, K, dtype=api.torch_dtype(dtype), device="cuda:0")
    api.topk(to_dev(hb, dtype), K, idx, dtype, vals=vals)
    torch.cuda.synchronize()
    got = idx.cpu().numpy()
    gv = to_bits(vals)
    for b in range(B):
        want = O.topk_indices(hb[b], K)
        assert np.array_equal(got[b], want)
        assert np.array_equal(gv[b], hb[b][want])


@pytest.mark.parametrize("dtype", ["f16", "bf16"])
@pytest.mark.parametrize("d", [504, 512, 520, 1024, 1032, 2048, 2056, 4096, 4104, 8192, 8200, 16384, 16392, 24576, 24584, 32768])
def test_topk_where_its_workgroup_changes(api, dtype, d):
    """Widths at which another number of waves, elements per lane or copies of the histogram takes over, the last lanes full
    or empty; vectors of 40 magnitudes (hundreds of ties at every threshold, the quota ending inside lanes) with zeros."""
    print(f"topk dtype={dtype} d={d}", flush=True)
    rng = np.random.default_rng(d)
    v = rng.choice(np.concatenate([[0.0], 2.0 ** rng.uniform(-9, 9, 39)]), (2, d)) * rng.choice([-1.0, 1.0], (2, d))
    hb = O.encode16(v, dtype)
    for K in (1, 2, d // 3, (3 * d) // 5, d - 1, d):
        idx = torch.full((2, K), -1, dtype=torch.int32, device="cuda:0")
        vals = torch.zeros(2, K, dtype=api.torch_dtype(dtype), device="cuda:0")
        api.topk(to_dev(hb, dtype), K, idx, dtype, vals=vals)
        torch.cuda.synchronize()
        for b in range(2):
            want = O.topk_indices(hb[b], K)
            assert np.array_equal(idx.cpu().numpy()[b], want), (K, b)
            assert np.array_equal(to_bits(vals)[b], hb[b][want]), (K, b)
        alone = torch.full((2, K), -1, dtype=torch.int32, device="cuda:0")   # a kernel of its own
        api.topk(to_dev(hb, dtype), K, alone, dtype)
        torch.cuda.synchronize()
        assert torch.equal(alone, idx), K


@pytest.mark.parametrize("dtype", ["f16", "bf16"])
def test_topk_ties_and_special_values(api, dtype):
    d = 4096
    rng = np.random.default_rng(3)
    cases = []
    cases.append(np.full(d, 0x3C00, np.uint16))                                     # all equal
    few = rng.choice(np.array([0x3C00, 0xBC00, 0x3800, 0x0000, 0x8000], np.uint16), d)   # five values, many ties
    cases.append(few)
    sp = O.encode16(rng.standard_normal(d), dtype)
    inf, ninf, nan = (0x7C00, 0xFC00, 0x7E01) if dtype == "f16" else (0x7F80, 0xFF80, 0x7FC1)
    sp[[5, 900, 4095]] = [inf, nan, ninf]
    sp[[17, 18]] = [0x0000, 0x8000]
    cases.append(sp)
    cases.append(np.repeat(O.encode16(rng.standard_normal(d // 4), dtype), 4))        # GQA-style repeats
    hb = np.stack(cases)
    for K in (1, 2, 1000, 2457, 4095, 4096):
        idx = torch.full((hb.shape[0], K), -1, dtype=torch.int32, device="cuda:0")
        api.topk(to_dev(hb, dtype), K, idx, dtype)
        torch.cuda.synchronize()
        got = idx.cpu().numpy()
        for b in range(hb.shape[0]):
            assert np.array_equal(got[b], O.topk_indices(hb[b], K)), (b, K)


@pytest.mark.parametrize("dtype", ["f16", "bf16"])
@pytest.mark.parametrize("B,d_in,d_out,K", [(1, 512, 1024, 256), (1, 512, 1000, 512), (3, 768, 1544, 300),
                                            (1, 64, 8, 1), (2, 2048, 6152, 1229), (1, 4096, 512, 4096)])
def test_sparse_gemv_matches_oracle(api, ws, dtype, B, d_in, d_out, K):
    print(f"sparse_gemv dtype={dtype} B={B} d_in={d_in} d_out={d_out} K={K}", flush=True)
    rng = np.random.default_rng(d_in + d_out + K)
    wb = O.encode16(synth.gaussian_weight(d_in, d_out, seed=d_out + K), dtype)
    hb, h = _heavy_vector(rng, B, d_in, dtype)
    idx = O.topk_batch(hb, K)
    y = torch.zeros(B, d_out, dtype=api.torch_dtype(dtype), device="cuda:0")
    dW = to_dev(wb, dtype)
    api.sparse_gemv(dW, to_dev(hb, dtype), torch.from_numpy(idx).cuda(), y, dtype, ws)
    torch.cuda.synchronize()
    W = O.decode16(wb, dtype)
    got = O.decode16(to_bits(y), dtype)
    for b in range(B):
        want = O.round16(O.sparse_project_gather(h[b], idx[b], W), dtype)   # stored 16-bit output
        stored_close(to_bits(y)[b], want, dtype, "sparse_gemv")
        assert rel_l2(got[b], O.round16(O.sparse_project_masked(h[b], idx[b], W), dtype)) <= REL_L2_TOL
    # unsorted index order is allowed and changes nothing but rounding order
    perm = np.stack([rng.permutation(idx[b]) for b in range(B)]).astype(np.int32)
    y2 = torch.zeros_like(y)
    api.sparse_gemv(dW, to_dev(hb, dtype), torch.from_numpy(perm).cuda(), y2, dtype, ws)
    torch.cuda.synchronize()
    for b in range(B):
        stored_close(to_bits(y2)[b], O.round16(O.sparse_project_gather(h[b], idx[b], W), dtype), dtype, "sparse_gemv, permuted indices")


def test_sparse_gemv_full_K_equals_dense_gemv_and_is_deterministic(api, ws):
    dtype, d_in, d_out = "f16", 1024, 2568
    rng = np.random.default_rng(5)
    wb = O.encode16(synth.gaussian_weight(d_in, d_out, seed=1), dtype)
    hb, h = _heavy_vector(rng, 2, d_in, dtype)
    ident = np.tile(np.arange(d_in, dtype=np.int32), (2, 1))
    dW, dh = to_dev(wb, dtype), to_dev(hb, dtype)
    y1 = torch.zeros(2, d_out, dtype=torch.float16, device="cuda:0")
    y2 = torch.zeros_like(y1)
    y3 = torch.zeros_like(y1)
    api.sparse_gemv(dW, dh, torch.from_numpy(ident).cuda(), y1, dtype, ws)
    api.dense_gemv(dW, dh, y2, dtype, ws)
    api.sparse_gemv(dW, dh, torch.from_numpy(ident).cuda(), y3, dtype, ws)
    torch.cuda.synchronize()
    assert np.array_equal(to_bits(y1), to_bits(y2))
    assert np.array_equal(to_bits(y1), to_bits(y3))
    want = O.round16(h @ O.decode16(wb, dtype), dtype)
    for b in range(2):
        stored_close(to_bits(y1)[b], want[b], dtype, "dense_gemv")


@pytest.mark.parametrize("variant,g_target,min_rows", [(0, 64, 4), (1, 2048, 1), (2, 256, 16), (0, 1024, 8),
                                                        (2, 512, 2), (1, 4096, 64)])
def test_sparse_gemv_every_launch_shape(api, variant, g_target, min_rows):
    """Each kernel shape variant and work split gives the same answer (within rounding order)."""
    dtype, d_in, d_out, K = "bf16", 1536, 3080, 777
    rng = np.random.default_rng(11)
    wb = O.encode16(synth.gaussian_weight(d_in, d_out, seed=2), dtype)
    hb, h = _heavy_vector(rng, 2, d_in, dtype)
    idx = O.topk_batch(hb, K)
    try:
        api.set_tuning(2, variant); api.set_tuning(0, g_target); api.set_tuning(1, min_rows)
        ws = api.workspace(2, d_in, d_out, K)
        y = torch.zeros(2, d_out, dtype=torch.bfloat16, device="cuda:0")
        api.sparse_gemv(to_dev(wb, dtype), to_dev(hb, dtype), torch.from_numpy(idx).cuda(), y, dtype, ws)
        torch.cuda.synchronize()
    finally:
        api.set_tuning(2, 0); api.set_tuning(0, 0); api.set_tuning(1, 8)
    W = O.decode16(wb, dtype)
    for b in range(2):
        stored_close(to_bits(y)[b], O.round16(O.sparse_project_gather(h[b], idx[b], W), dtype), dtype, "sparse_gemv")


@pytest.mark.parametrize("dtype", ["f16", "bf16"])
@pytest.mark.parametrize("B", [2, 4, 5, 16, 17, 33])
def test_batched_sparse_gemv_per_token_index_sets(api, dtype, B):
    """Batched variant: independent index sets per token; 2-4 tokens take the FMA kernel, 5-32 the
    matrix-core kernel, more than 32 several token groups.  Row count not a multiple of the 16-row
    tile, output width with a ragged last strip."""
    d_in, d_out, K = 1032, 1544, 413
    print(f"batched sparse_gemv dtype={dtype} B={B}", flush=True)
    rng = np.random.default_rng(1000 + B)
    wb = O.encode16(synth.gaussian_weight(d_in, d_out, seed=3), dtype)
    hb, h = _heavy_vector(rng, B, d_in, dtype)
    idx = O.topk_batch(hb, K)
    ws = api.workspace(B, d_in, d_out, K)
    y = torch.full((B, d_out), 7.0, dtype=api.torch_dtype(dtype), device="cuda:0")
    api.sparse_gemv(to_dev(wb, dtype), to_dev(hb, dtype), torch.from_numpy(idx).cuda(), y, dtype, ws)
    torch.cuda.synchronize()
    W = O.decode16(wb, dtype)
    for b in range(B):
        want = O.round16(O.sparse_project_gather(h[b], idx[b], W), dtype)
        stored_close(to_bits(y)[b], want, dtype, f"batched sparse_gemv token {b}")
    # a second call on the same workspace gives the same bits (counters were left at zero)
    y2 = torch.zeros_like(y)
    api.sparse_gemv(to_dev(wb, dtype), to_dev(hb, dtype), torch.from_numpy(idx).cuda(), y2, dtype, ws)
    torch.cuda.synchronize()
    assert np.array_equal(to_bits(y), to_bits(y2))


@pytest.mark.parametrize("dtype", ["f16", "bf16"])
@pytest.mark.parametrize("B,d", [(2, 520), (8, 2048), (16, 4096), (32, 1096)])
def test_batched_rotate_matches_oracle(api, dtype, B, d):
    print(f"batched rotate dtype={dtype} B={B} d={d}", flush=True)
    rng = np.random.default_rng(200 + d + B)
    qb = O.encode16(synth.planted_basis(d, seed=d + 1), dtype)
    xb, x = _heavy_vector(rng, B, d, dtype)
    ws = api.workspace(B, d, d, d)
    h = torch.zeros(B, d, dtype=api.torch_dtype(dtype), device="cuda:0")
    api.rotate(to_dev(xb, dtype), to_dev(qb, dtype), h, dtype, ws)
    torch.cuda.synchronize()
    want = O.round16(O.rotate(x, O.decode16(qb, dtype)), dtype)
    for b in range(B):
        stored_close(to_bits(h)[b], want[b], dtype, f"batched rotate token {b}")


def test_config0_single_linear_by_its_recipe(api, ws):
    """The smallest benchmark configuration end to end through the three calls: a single linear layer
    512 x 1024, fp16, W ~ N(0, 0.02^2); tokens x = (z * s) U^T with s_i = i^-0.8 and 4 outlier channels
    x 20; Q = PCA of 2048 calibration tokens drawn the same way; W' = Q^T W rounded once.
    rotate -> Top-K (K = 256) -> column-sparse product, each stage against the oracle on the GPU's own
    stage input; and at K = d the result equals the dense product x W with the UNFOLDED weight
    (computational invariance, Sec. 3.2), to the accuracy of 16-bit storage."""
    d, d_out, K, dtype = 512, 1024, 256, "f16"
    seed = synth.seed_for(0, 0)
    src = synth.activation_source(d, seed)
    Xc = src.draw(2048, seed + 1)
    Q, lam = O.pca_rotation(O.second_moment(Xc))
    W = synth.gaussian_weight(d, d_out, seed=seed + 100).astype(np.float64)
    qb, wb = O.encode16(Q, dtype), O.encode16(O.fold_input_side(Q, W), dtype)
    xb = O.encode16(src.draw(1, seed + 5), dtype)
    x = O.decode16(xb, dtype)
    td = api.torch_dtype(dtype)
    h = torch.zeros(1, d, dtype=td, device="cuda:0")
    api.rotate(to_dev(xb, dtype), to_dev(qb, dtype), h, dtype, ws)
    torch.cuda.synchronize()
    stored_close(to_bits(h)[0], O.round16(O.rotate(x[0], O.decode16(qb, dtype)), dtype), dtype, "h = x Q")
    hb = to_bits(h)
    hv = O.decode16(hb, dtype)
    for Kc in (K, d):
        idx = torch.full((1, Kc), -1, dtype=torch.int32, device="cuda:0")
        api.topk(h, Kc, idx, dtype)
        torch.cuda.synchronize()
        want_idx = O.topk_indices(hb[0], Kc)
        assert np.array_equal(idx.cpu().numpy()[0], want_idx)
        y = torch.zeros(1, d_out, dtype=td, device="cuda:0")
        api.sparse_gemv(to_dev(wb, dtype), h, idx, y, dtype, ws)
        torch.cuda.synchronize()
        stored_close(to_bits(y)[0], O.round16(O.sparse_project_gather(hv[0], want_idx, O.decode16(wb, dtype)), dtype),
                     dtype, f"y at K = {Kc}")
        if Kc == d:
            dense = x[0] @ W        # fp64, unfolded weight, unrotated token
            got = O.decode16(to_bits(y), dtype)[0]
            # three 16-bit roundings separate the two (Q, h, W'): each is 2^-11 relative per entry
            assert rel_l2(got, dense) <= 3e-3


@pytest.mark.parametrize("dtype", ["f16", "bf16"])
@pytest.mark.parametrize("B,d_in,d_out", [(17, 8, 8), (32, 40, 136), (31, 1000, 4096), (32, 4120, 1544), (17, 1032, 5128), (33, 72, 33032), (17, 520, 33024),
                                          (48, 4120, 1032)])
def test_more_than_16_tokens_in_both_strip_widths(api, dtype, B, d_in, d_out):
    """Groups of 32 tokens, and (17 .. 32 tokens, small weights) two groups of 16 instead: fewer rows than one tile, ragged
    rows and columns, a last group with one or 16 tokens, strips of 128 columns and (more than 32768 outputs) of 256; and wide outputs on a workspace that only
    holds the partial sums of 128-column strips."""
    print(f"B={B} d_in={d_in} d_out={d_out} {dtype}", flush=True)
    rng = np.random.default_rng(1700 + B)
    xb = O.encode16(rng.standard_normal((B, d_in)), dtype)
    wb = O.encode16(synth.gaussian_weight(d_in, d_out, B), dtype)
    want = O.decode16(xb, dtype) @ O.decode16(wb, dtype)
    x, W = to_dev(xb, dtype), to_dev(wb, dtype)
    sizes = [api.workspace_bytes(B, d_in, d_out, d_in)]
    if d_out > 32768:
        sizes.append((1 << 20) + (B + 31) // 32 * 32 * ((d_out + 127) // 128) * 128 * 4)
    outs = []
    for nbytes in sizes:
        w = api.Workspace(nbytes)
        y = torch.full((B, d_out), 7.0, dtype=x.dtype, device="cuda:0")
        for _ in range(2):                                    # the arrival counters are left at zero
            api.dense_gemv(W, x, y, dtype, w)
        torch.cuda.synchronize()
        stored_close(to_bits(y), want, dtype, f"workspace {nbytes}")
        outs.append(to_bits(y))
    assert all(rel_l2(O.decode16(o, dtype), O.decode16(outs[0], dtype)) <= REL_L2_TOL for o in outs)


@pytest.mark.parametrize("dtype", ["f16", "bf16"])
@pytest.mark.parametrize("B,d_in,d_out", [(17, 8, 8), (33, 72, 136), (33, 1000, 4096), (32, 4120, 1544), (40, 1040, 16648), (33, 2056, 16520),
                                          (31, 2120, 4104), (32, 2048, 4096), (32, 8192, 6144), (17, 520, 33032), (33, 1032, 33032)])
def test_a_tokens_bits_do_not_depend_on_its_batch(api, dtype, B, d_in, d_out):
    """More than 16 tokens run in kernels of their own (groups of 32, of eight or four waves, strips of 128 or 256
    columns); they add a token's products in the order of the kernel for up to 16, so every token's result has the bits
    that it has in a batch of 16.  Sizes: runs of rows that are empty, end inside a tile or differ in length, with and
    without a hand-off between workgroups."""
    print(f"B={B} d_in={d_in} d_out={d_out} {dtype}", flush=True)
    rng = np.random.default_rng(1900 + B + d_in)
    x = to_dev(O.encode16(rng.standard_normal((B, d_in)), dtype), dtype)
    W = to_dev(O.encode16(synth.gaussian_weight(d_in, d_out, B), dtype), dtype)
    w = api.workspace(B, d_in, d_out, d_in)
    y = torch.zeros(B, d_out, dtype=x.dtype, device="cuda:0")
    api.dense_gemv(W, x, y, dtype, w)
    for first in list(range(0, B - 16, 16)) + [B - 16]:
        part = torch.zeros(16, d_out, dtype=x.dtype, device="cuda:0")
        api.dense_gemv(W, x[first:first + 16].contiguous(), part, dtype, w)
        torch.cuda.synchronize()
        assert torch.equal(part.view(torch.int16), y[first:first + 16].view(torch.int16)), first


def test_many_workgroups_per_strip_of_a_wide_output(api):
    """Asked for more workgroups than strips, a wide output keeps 128-column strips, whose workgroups hand over to each
    other (strips of 256 columns have one workgroup each)."""
    rng = np.random.default_rng(2000)
    B, d_in, d_out, dtype = 33, 1000, 33032, "f16"
    xb = O.encode16(rng.standard_normal((B, d_in)), dtype)
    wb = O.encode16(synth.gaussian_weight(d_in, d_out, B), dtype)
    x, W, y = to_dev(xb, dtype), to_dev(wb, dtype), torch.zeros(B, d_out, dtype=torch.float16, device="cuda:0")
    api.set_tuning(0, 1024)
    try:
        w = api.workspace(B, d_in, d_out, d_in)
        for _ in range(2):                                    # the arrival counters are left at zero
            y.fill_(7.0)
            api.dense_gemv(W, x, y, dtype, w)
            torch.cuda.synchronize()
            stored_close(to_bits(y), O.decode16(xb, dtype) @ O.decode16(wb, dtype), dtype, "wide output")
    finally:
        api.set_tuning(0, 0)


@pytest.mark.parametrize("B", [2, 17])
def test_inputs_of_2_to_the_25_channels_stay_on_the_matrix_cores(api, B):
    """32 tokens of 2^25 channels are 2 GiB of coefficients, past the 32-bit offsets of the kernel for groups of 32: the one
    for 16 tokens takes them, on the workspace of its 256 workgroups (the vector-unit kernel would need 8192)."""
    print(f"B={B} d_in=2^25", flush=True)
    d_in, d_out, dtype = 1 << 25, 8, "f16"
    g = torch.Generator(device="cuda:0").manual_seed(B)
    x = torch.randn(B, d_in, generator=g, device="cuda:0", dtype=torch.float16)
    W = torch.randn(d_in, d_out, generator=g, device="cuda:0", dtype=torch.float16)
    y = torch.zeros(B, d_out, dtype=torch.float16, device="cuda:0")
    ws = api.Workspace((1 << 20) + (B + 15) // 16 * 16 * 256 * 128 * 4)
    api.dense_gemv(W, x, y, dtype, ws)
    torch.cuda.synchronize()
    W64 = W.double()
    want = torch.stack([x[b].double() @ W64 for b in range(B)]).cpu().numpy()
    stored_close(to_bits(y), want, dtype, "2^25 channels")


@pytest.mark.parametrize("d_in", [8, 4096, 4104, 64 * 4096 + 8, (1 << 23) + 4096 + 8])
def test_masked_coefficients_of_every_slice(api, d_in):
    """Several tokens with unsorted index lists: the masked coefficients are written in slices of 4096 channels, of more than
    that past 64 slices, and of 131072 past 2^23 channels.  The result has the bits of the dense product of the masked
    tokens."""
    print(f"d_in={d_in}", flush=True)
    B, d_out, dtype = 3, 8, "f16"
    K = max(1, d_in * 3 // 7)
    g = torch.Generator(device="cuda:0").manual_seed(d_in)
    h = torch.randn(B, d_in, generator=g, device="cuda:0", dtype=torch.float16)
    W = torch.randn(d_in, d_out, generator=g, device="cuda:0", dtype=torch.float16)
    idx = torch.stack([torch.randperm(d_in, generator=g, device="cuda:0")[:K] for _ in range(B)])
    masked = torch.zeros_like(h).scatter_(1, idx, h.gather(1, idx))
    ws = api.workspace(B, d_in, d_out, K)
    got, want = (torch.zeros(B, d_out, dtype=torch.float16, device="cuda:0") for _ in range(2))
    api.sparse_gemv(W, h, idx.int().contiguous(), got, dtype, ws)
    api.dense_gemv(W, masked, want, dtype, ws)
    torch.cuda.synchronize()
    assert torch.equal(got.view(torch.int16), want.view(torch.int16))
