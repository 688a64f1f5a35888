"""GPU parity, through the C ABI, of the 4-bit-weight projection (quantiser: codes and scales equal
to the oracle's bit for bit; projection within 2e-3 relative L2 of the oracle's rounded output) and of
the magnitude-threshold sparsifier (indices and counts equal)."""
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
    return api.workspace(4, 32768, 32768, 32768)


def _heavy(rng, B, d, dtype):
    v = rng.standard_normal((B, d)) * (np.arange(1, d + 1) ** -0.6)[None, :]
    v[:, rng.choice(d, min(4, d), replace=False)] *= 20
    bits = O.encode16(v, dtype)
    return bits, O.decode16(bits, dtype)


def _dev_w4(codes, sbits, dtype):
    packed = O.pack_w4(codes)
    return torch.from_numpy(packed.view(np.int32)).cuda(), to_dev(sbits, dtype)


@pytest.mark.parametrize("dtype", ["f16", "bf16"])
@pytest.mark.parametrize("d_in,d_out", [(37, 328), (64, 1024), (5, 8), (33, 704), (130, 1160)])
def test_quantiser_equals_oracle_bit_for_bit(api, dtype, d_in, d_out):
    print(f"quantize_w4 dtype={dtype} {d_in}x{d_out}", flush=True)
    wb = O.encode16(synth.gaussian_weight(d_in, d_out, 21 + d_out), dtype)
    wb[0, :min(128, d_out)] = 0                                   # a zero group
    Wq, sc = api.quantize_w4(to_dev(wb, dtype), dtype)
    torch.cuda.synchronize()
    codes, sbits = O.quantize_rtn_w4(O.decode16(wb, dtype), dtype)
    assert np.array_equal(to_bits(sc), sbits)
    assert np.array_equal(Wq.cpu().numpy().view(np.uint32), O.pack_w4(codes))


@pytest.fixture(params=[32768, 2048], ids=["narrow", "wide"])
def w4_geometry(api, request):
    """The 4-bit kernel's two geometries: 512-column strips with dword loads, and 2048-column strips
    with 16-byte loads (by default only for outputs of 32768 columns or more; forced here)."""
    api.set_tuning(7, request.param)
    yield request.param
    api.set_tuning(7, 32768)


@pytest.mark.parametrize("dtype", ["f16", "bf16"])
@pytest.mark.parametrize("B,d_in,d_out,K", [(1, 512, 1024, 256), (3, 1096, 1160, 700), (1, 64, 8, 64), (2, 2048, 4096, 1),
                                            (2, 520, 2080, 300), (1, 4096, 2048, 4096), (1, 1000, 6144, 613)])
def test_w4_projection_matches_oracle(api, ws, w4_geometry, dtype, B, d_in, d_out, K):
    print(f"sparse_gemv_w4 dtype={dtype} B={B} {d_in}x{d_out} K={K} geometry={w4_geometry}", flush=True)
    rng = np.random.default_rng(300 + d_in + K)
    codes, sbits = O.quantize_rtn_w4(synth.gaussian_weight(d_in, d_out, 31 + d_in), dtype)
    Wq, sc = _dev_w4(codes, sbits, dtype)
    hb, h = _heavy(rng, B, d_in, dtype)
    idx = O.topk_batch(hb, K)
    y = torch.zeros(B, d_out, dtype=api.torch_dtype(dtype), device="cuda:0")
    api.sparse_gemv_w4(Wq, sc, to_dev(hb, dtype), torch.from_numpy(idx).cuda(), y, dtype, ws)
    torch.cuda.synchronize()
    got = O.decode16(to_bits(y), dtype)
    for b in range(B):
        want = O.round16(O.sparse_project_w4(h[b], idx[b], codes, sbits, dtype), dtype)
        assert rel_l2(got[b], want) <= REL_L2_TOL
    # all rows, no index list
    api.sparse_gemv_w4(Wq, sc, to_dev(hb, dtype), None, y, dtype, ws)
    torch.cuda.synchronize()
    got = O.decode16(to_bits(y), dtype)
    deq = O.dequantize_w4(codes, sbits, dtype)
    for b in range(B):
        assert rel_l2(got[b], O.round16(h[b] @ deq, dtype)) <= REL_L2_TOL
    # same call twice: same bits
    y2 = torch.zeros_like(y)
    api.sparse_gemv_w4(Wq, sc, to_dev(hb, dtype), None, y2, dtype, ws)
    torch.cuda.synchronize()
    assert torch.equal(y.view(torch.int16), y2.view(torch.int16))


@pytest.mark.parametrize("dtype", ["f16", "bf16"])
@pytest.mark.parametrize("per_wave", [1, 15, 16, 17, 32, 33, 48, 49, 64, 65, 80, 81])
def test_w4_row_batches_in_flight(api, ws, dtype, per_wave):
    """One workgroup per strip with `per_wave` rows for each of its waves (the last one fewer): every way the pipeline of
    16-row batches can begin and end, against one launch for many tokens, which takes the loop of single batches (the sums
    are formed in the same order: same bits), and against the oracle.  The second strip holds 8 columns."""
    d_in, d_out, K, many = 704, 520, 8 * per_wave - 3, 200
    print(f"sparse_gemv_w4 batches dtype={dtype} per_wave={per_wave}", flush=True)
    rng = np.random.default_rng(per_wave)
    codes, sbits = O.quantize_rtn_w4(synth.gaussian_weight(d_in, d_out, 31), dtype)
    Wq, sc = _dev_w4(codes, sbits, dtype)
    hb, h = _heavy(rng, 1, d_in, dtype)
    idx = O.topk_batch(hb, K)
    api.set_tuning(1, 1 << 20)
    try:
        ys = []
        for B in (1, many):
            y = torch.zeros(B, d_out, dtype=api.torch_dtype(dtype), device="cuda:0")
            api.sparse_gemv_w4(Wq, sc, to_dev(np.repeat(hb, B, 0), dtype), torch.from_numpy(np.repeat(idx, B, 0)).cuda(), y, dtype,
                               ws if B == 1 else api.workspace(B, d_in, d_out, K))
            torch.cuda.synchronize()
            ys.append(to_bits(y))
    finally:
        api.set_tuning(1, 112)
    assert (ys[1] == ys[0][0]).all()
    want = O.round16(O.sparse_project_w4(h[0], idx[0], codes, sbits, dtype), dtype)
    assert rel_l2(O.decode16(ys[0], dtype)[0], want) <= REL_L2_TOL


def test_w4_projection_full_size_gate_up(api, ws, w4_geometry):
    """gate|up of the 7B-shaped layer (4096 x 22016, 40 % sparsity) in the launch shape the bench times."""
    dtype, d_in, d_out, K = "f16", 4096, 22016, 2458
    print("sparse_gemv_w4 full size", flush=True)
    rng = np.random.default_rng(77)
    wb = O.encode16(synth.gaussian_weight(d_in, d_out, 41), dtype)
    Wq, sc = api.quantize_w4(to_dev(wb, dtype), dtype)          # checked bit for bit above; reused here as input
    torch.cuda.synchronize()
    codes = O.unpack_w4(Wq.cpu().numpy().view(np.uint32))
    sbits = to_bits(sc)
    rows = np.sort(rng.choice(d_in, 16, replace=False))
    c_or, s_or = O.quantize_rtn_w4(O.decode16(wb[rows], dtype), dtype)
    assert np.array_equal(codes[rows], c_or) and np.array_equal(sbits[rows], s_or)
    hb, h = _heavy(rng, 1, d_in, dtype)
    idx = O.topk_batch(hb, K)
    y = torch.zeros(1, d_out, dtype=torch.float16, device="cuda:0")
    api.sparse_gemv_w4(Wq, sc, to_dev(hb, dtype), torch.from_numpy(idx).cuda(), y, dtype, ws)
    torch.cuda.synchronize()
    want = O.round16(O.sparse_project_w4(h[0], idx[0], codes, sbits, dtype), dtype)
    assert rel_l2(O.decode16(to_bits(y), dtype)[0], want) <= REL_L2_TOL


def test_w4_wide_geometry_at_the_shape_that_selects_it(api):
    """gate|up of the LLaMA2-70B-shaped layer: 8192 x 57344, K = 4915 (40 % sparsity), bf16 -- the one
    benchmark shape whose output is wide enough for the 2048-column geometry to be chosen by the library
    itself (no tuning override).  Weights are drawn and quantised on the device (the quantiser is checked
    bit for bit above, and again here on sampled rows); the projection is checked on sampled output
    columns that span several strips, the ragged last one included, against the oracle's product over
    the same codes and scales."""
    dtype, d_in, d_out, K = "bf16", 8192, 57344, 4915
    print("sparse_gemv_w4 8192 x 57344, default geometry", flush=True)
    gen = torch.Generator(device="cuda:0")
    gen.manual_seed(1299)
    Wd = (torch.randn(d_in, d_out, generator=gen, device="cuda:0", dtype=torch.float32) * 0.02).to(torch.bfloat16)
    Wq, sc = api.quantize_w4(Wd, dtype)
    torch.cuda.synchronize()
    rng = np.random.default_rng(91)
    rows = np.sort(rng.choice(d_in, 8, replace=False))
    c_or, s_or = O.quantize_rtn_w4(O.decode16(to_bits(Wd[torch.from_numpy(rows).cuda()]), dtype), dtype)
    codes_rows = O.unpack_w4(Wq[torch.from_numpy(rows).cuda()].cpu().numpy().view(np.uint32))
    assert np.array_equal(codes_rows, c_or) and np.array_equal(to_bits(sc[torch.from_numpy(rows).cuda()]), s_or)
    del Wd
    hb, h = _heavy(rng, 1, d_in, dtype)
    idx = O.topk_batch(hb, K)
    ws = api.workspace(1, d_in, d_out, K)
    y = torch.zeros(1, d_out, dtype=torch.bfloat16, device="cuda:0")
    api.sparse_gemv_w4(Wq, sc, to_dev(hb, dtype), torch.from_numpy(idx).cuda(), y, dtype, ws)
    torch.cuda.synchronize()
    # sampled groups of 128 columns (one scale group each): first, last, strip boundaries, random ones
    groups = sorted({0, 15, 16, 17, d_out // 128 - 1, *rng.choice(d_out // 128, 12, replace=False).tolist()})
    kept = torch.from_numpy(idx[0].astype(np.int64)).cuda()
    Wq_k, sc_k = Wq[kept], sc[kept]                 # the kept rows' codes and scales
    got = O.decode16(to_bits(y), dtype)[0]
    for gidx in groups:
        c0 = gidx * 128
        codes_g = O.unpack_w4(Wq_k[:, c0 // 8:(c0 + 128) // 8].contiguous().cpu().numpy().view(np.uint32))   # [K, 128]
        sb_g = to_bits(sc_k[:, gidx:gidx + 1].contiguous())                                                  # [K, 1]
        want = O.round16(O.sparse_project_w4(h[0][idx[0]], np.arange(K), codes_g, sb_g, dtype), dtype)
        stored_close(to_bits(y)[0][c0:c0 + 128], want, dtype, f"columns {c0}..{c0 + 127}")
    assert np.isfinite(got).all()


@pytest.mark.parametrize("dtype", ["f16", "bf16"])
@pytest.mark.parametrize("B,d", [(1, 8), (3, 1096), (2, 4096), (1, 11008), (1, 32768)])
def test_threshold_select_equals_oracle(api, dtype, B, d):
    print(f"threshold_select dtype={dtype} B={B} d={d}", flush=True)
    rng = np.random.default_rng(500 + d)
    hb, h = _heavy(rng, B, d, dtype)
    cal = _heavy(rng, 8, d, dtype)[1]
    idx = torch.full((B, d), -1, dtype=torch.int32, device="cuda:0")
    cnt = torch.full((B,), -1, dtype=torch.int32, device="cuda:0")
    eps_list = [np.float32(O.calibrate_threshold(cal, p)) for p in (0.25, 0.4, 0.5)]
    eps_list += [np.float32(0.0), np.float32(1e30), np.float32(abs(h[0, d // 2]))]     # the last one: an exact tie
    for eps in eps_list:
        idx.fill_(-1)
        api.threshold_select(to_dev(hb, dtype), float(eps), idx, cnt, dtype)
        torch.cuda.synchronize()
        gi, gc = idx.cpu().numpy(), cnt.cpu().numpy()
        for b in range(B):
            want = O.threshold_indices(h[b], float(eps))
            assert gc[b] == want.size
            assert np.array_equal(gi[b, :want.size], want)
            assert np.all(gi[b, want.size:] == -1)                # nothing written past the count


def test_threshold_then_projection_is_the_masked_product(api, ws):
    """S_eps(h) W with the kept count read back: the variable-K comparison path (Eq. 3-5)."""
    dtype, d, d_out = "f16", 1096, 1160
    rng = np.random.default_rng(900)
    wb = O.encode16(synth.gaussian_weight(d, d_out, 51), dtype)
    W = O.decode16(wb, dtype)
    hb, h = _heavy(rng, 1, d, dtype)
    eps = np.float32(O.calibrate_threshold(_heavy(rng, 8, d, dtype)[1], 0.4))
    idx = torch.zeros(1, d, dtype=torch.int32, device="cuda:0")
    cnt = torch.zeros(1, dtype=torch.int32, device="cuda:0")
    api.threshold_select(to_dev(hb, dtype), float(eps), idx, cnt, dtype)
    K = int(cnt.item())
    assert 0 < K < d
    y = torch.zeros(1, d_out, dtype=torch.float16, device="cuda:0")
    api.sparse_gemv(to_dev(wb, dtype), to_dev(hb, dtype), idx[:, :K].contiguous(), y, dtype, ws)
    torch.cuda.synchronize()
    masked = np.where(np.abs(h[0]) > float(eps), h[0], 0.0)
    assert rel_l2(O.decode16(to_bits(y), dtype)[0], O.round16(masked @ W, dtype)) <= REL_L2_TOL


@pytest.mark.parametrize("dtype", ["f16", "bf16"])
@pytest.mark.parametrize("d_in,d_out", [(1, 8), (15, 512), (17, 520), (33, 1032)])
def test_quantiser_on_ties_and_extreme_groups(api, dtype, d_in, d_out):
    """Quotients that are exact half-integers (the rounding decides), groups of zeros, and groups whose scale is at
    the ends of the storage type's range; row counts around the 16 rows of a workgroup."""
    rng = np.random.default_rng(41 * d_in + d_out)
    k = rng.integers(-14, 15, size=(d_in, d_out)).astype(np.float64)          # w / s = k / 2: every odd k is a tie
    ng = (d_out + 127) // 128
    exps = rng.integers(-10, 4, size=(d_in, ng)) if dtype == "f16" else rng.integers(-118, 100, size=(d_in, ng))
    for g in range(ng):
        k[:, g * 128] = 14.0                                                    # the scale is 2^e exactly
        k[:, g * 128:(g + 1) * 128] *= 2.0 ** exps[:, g:g + 1] / 2
    k[d_in // 2, :min(128, d_out)] = 0.0
    wb = O.encode16(k, dtype)
    codes, sbits = O.quantize_rtn_w4(O.decode16(wb, dtype), dtype)
    q, s = api.quantize_w4(to_dev(wb, dtype), dtype)
    torch.cuda.synchronize()
    assert np.array_equal(q.cpu().numpy().view(np.uint32), O.pack_w4(codes))
    assert np.array_equal(to_bits(s), sbits)


@pytest.mark.parametrize("dtype", ["f16", "bf16"])
def test_quantiser_on_nan_and_infinite_groups(api, dtype):
    """A NaN does not count for its group's scale; its code is 8 where the scale is zero, else 0 (the lowest).  An infinite
    group has an infinite scale: code 0 for the infinities themselves, 8 for the rest."""
    rng = np.random.default_rng(47)
    W = rng.standard_normal((6, 512))
    W[:, :128] = 0.0
    W[0, 5] = W[0, 127] = W[3, 64] = np.nan                       # zeros and NaN: scale 0
    W[1, 128:256] = np.nan                                        # nothing but NaN: scale 0
    W[2, 256:384:3] = np.nan                                      # NaN among numbers
    W[4, 384], W[4, 390], W[4, 400] = np.inf, -np.inf, np.nan
    wb = np.where(np.isnan(W), np.uint16(0x7E00 if dtype == "f16" else 0x7FC0), O.encode16(np.nan_to_num(W, posinf=np.inf, neginf=-np.inf), dtype))
    w64 = O.decode16(wb, dtype)
    finite = np.where(np.isfinite(w64), w64, 0.0)
    codes, sbits = O.quantize_rtn_w4(finite, dtype)
    codes = np.where(np.isnan(w64) & (np.repeat(O.decode16(sbits, dtype), 128, axis=1) > 0), 0, codes)
    codes[4, 384:] = 8
    codes[4, [384, 390, 400]] = 0
    sbits[4, 3] = O.encode16(np.array([np.inf]), dtype)[0]
    q, s = api.quantize_w4(to_dev(wb.astype(np.uint16), dtype), dtype)
    torch.cuda.synchronize()
    assert np.array_equal(to_bits(s), sbits)
    assert np.array_equal(q.cpu().numpy().view(np.uint32), O.pack_w4(codes.astype(np.uint8)))


@pytest.mark.parametrize("dtype", ["f16", "bf16"])
def test_quantiser_on_ties_of_scales_with_rounded_reciprocals(api, dtype):
    """Scales S 2^e with S odd: 1 / S is not representable, so w times the rounded reciprocal misses some of the exact
    half-integers w / s = k / 2 and rounds them to the other neighbour (worked out here in 32 bits: the inputs hold such
    pairs).  The codes are those of the division."""
    bits, exps = (11, range(-12, 4)) if dtype == "f16" else (8, range(-90, 91, 12))
    rng = np.random.default_rng(53)
    odd = np.arange(3, 2 ** bits // 7, 2)                         # 7 S, the group's largest value, is representable
    S = np.tile(odd, 3)
    W = np.zeros((len(S), 128))
    missed = 0
    for r, s in enumerate(S):
        ks = np.array([k for k in range(-13, 14) if abs(k) * s < 2 ** bits])
        k = rng.choice(ks, 128)
        k[:len(ks)] = ks                                          # every tie of this scale that is representable
        w = k * (s / 2.0)
        plain = np.rint((w.astype(np.float32) * (np.float32(1.0) / np.float32(s))).astype(np.float32))
        missed += int((plain != np.rint(k / 2.0)).sum())
        w[127] = 7.0 * s
        W[r] = w * 2.0 ** rng.choice(exps)
    assert missed > 0
    wb = O.encode16(W, dtype)
    assert np.array_equal(O.decode16(wb, dtype), W)               # nothing was rounded on the way in
    codes, sbits = O.quantize_rtn_w4(W, dtype)
    q, sc = api.quantize_w4(to_dev(wb, dtype), dtype)
    torch.cuda.synchronize()
    assert np.array_equal(to_bits(sc), sbits)
    assert np.array_equal(q.cpu().numpy().view(np.uint32), O.pack_w4(codes))
