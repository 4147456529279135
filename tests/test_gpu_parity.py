"""GPU parity: the HIP path (through the C ABI) against the fp64 CPU oracle.

Codes and norms: bit-exact except counted decision-boundary ties.
Attention: max over (sequence, query head) of ||o_gpu - o_ref||_inf / ||o_ref||_inf <= 2e-3.
"""
import math
import sys

import numpy as np
import pytest

from oracle import blockgtq_oracle as o
from paper_2606_24033_amd import synth
from tests import _parity as P

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module", autouse=True)
def _require_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2606_24033_amd import blockgtq as bg
    bg.lib()  # loud failure if the library is missing


def bgm():
    from paper_2606_24033_amd import blockgtq as bg
    return bg


def log(*a):
    print(*a, flush=True)
    sys.stdout.flush()


def to_dev(x, dtype):
    t = torch.from_numpy(np.ascontiguousarray(x, dtype=np.float32))
    return t.to(device="cuda", dtype=torch.bfloat16 if dtype == "bf16" else torch.float32).contiguous()


def build(st):
    bg = bgm()
    assert np.array_equal(st.bits, st.bits_oracle), "library and oracle allocations differ"
    layout = bg.Layout(st.cfg, st.bits, synth.flat_rot_k(st.rot_k), st.rot_v)
    cache = bg.Cache(st.cfg)
    return layout, cache


def append(st, layout, cache, layer, kv_list, write_pos):
    """kv_list[seq][head] = (k [n,128], v [n,128]) -> one quantize_append call."""
    bg = bgm()
    B, H = st.cfg.batch, st.cfg.n_kv_heads
    n = kv_list[0][0][0].shape[0]
    K = np.zeros((B, n, H, 128), np.float32)
    V = np.zeros((B, n, H, 128), np.float32)
    for b in range(B):
        for h in range(H):
            K[b, :, h], V[b, :, h] = kv_list[b][h]
    wp = torch.tensor(write_pos, dtype=torch.int32, device="cuda")
    bg.blockgtq_quantize_append(st.cfg, layout, layer, to_dev(K, st.dtype), to_dev(V, st.dtype), wp, cache,
                                host_write_pos=list(write_pos))


def check_cache(st, cache, layer, seq, head, rows, T, stats, what):
    bits = st.bits_oracle[layer, head]
    widths = P.stream_widths(bits)
    words = cache.k_codes[layer, seq, head, :T].cpu().numpy().view(np.uint32)
    if not np.array_equal(words, rows.kwords[:T]):
        P.compare_codes(P.read_fields(words, widths), rows.kcodes[:T], rows.kz[:T], widths, P.group_dims(bits),
                        stats, what + " K")
    else:
        stats.codes += rows.kcodes[:T].size
    ng = rows.knorms.shape[1]
    S = ng + (ng & 1)   # token-major radii, n_g rounded up to even per token
    kn = cache.k_norms[layer, seq, head, :T * S].cpu().numpy().reshape(T, S)[:, :ng]
    P.compare_norms(kn, rows.knorms[:T], rows.kexact[:T], 128, stats, what + " K norms")
    vt = cache.v_codes[layer, seq, head].cpu().numpy().view(np.uint32)
    vc = P.read_value_codes(vt, st.cfg.v_bits, T)
    P.compare_codes(vc, rows.vcodes[:T], rows.vz[:T], np.full(128, st.cfg.v_bits), np.full(128, 128), stats,
                    what + " V")
    vn = cache.v_norms[layer, seq, head, :T].cpu().numpy()
    P.compare_norms(vn, rows.vnorms[:T], rows.vexact[:T], 128, stats, what + " V norms")


def concat_rows(a, b):
    return P.OracleRows(*[np.concatenate([x, y]) for x, y in zip(vars(a).values(), vars(b).values())])


# ----------------------------------------------------------------------------

def test_toy_single_head_end_to_end():
    """1 layer, 1 KV head, G = 4, d_h = 128, base 1e4, 2048 fp32 rows, K3V2,
    allocator on 256 calibration keys; append row 2048, attend 2049 rows."""
    bg = bgm()
    st = P.make_setup(1, 1, 1, 1, 4, 2112, 192, 2, 1e4, "fp32", n_cal=256)
    layout, cache = build(st)
    k, v = P.keys_values(st, 0, 0, 0, 2049)
    append(st, layout, cache, 0, [[(k[:2048], v[:2048])]], [0])
    append(st, layout, cache, 0, [[(k[2048:], v[2048:])]], [2048])
    rows = P.oracle_rows(st, 0, 0, k, v)
    stats = P.Stats()
    check_cache(st, cache, 0, 0, 0, rows, 2049, stats, "toy")
    log("toy ties", vars(stats))
    q = synth.cast(synth.queries(1, 0, 0, 2048, 4, 1e4), "fp32")
    ctx = torch.tensor([2049], dtype=torch.int32, device="cuda")
    for ns in (0, 1, 5):
        out = bg.blockgtq_decode_attn(st.cfg, layout, 0, to_dev(q[None], "fp32"), ctx, 2049, cache, n_splits=ns)
        ref = P.oracle_attention(st, 0, 0, q, rows, 2049)
        err = P.rel_err(out[0].cpu().numpy().astype(np.float64), ref)
        log("toy n_splits", ns, "rel err", err)
        assert err <= 2e-3
    # fp16 comparator against the definition on fp16-rounded K/V
    k16 = torch.zeros((1, 1, 1, st.cfg.capacity, 128), dtype=torch.float16, device="cuda")
    v16 = torch.zeros_like(k16)
    k16[0, 0, 0, :2049] = torch.from_numpy(k.astype(np.float32)).half().cuda()
    v16[0, 0, 0, :2049] = torch.from_numpy(v.astype(np.float32)).half().cuda()
    out16 = bg.blockgtq_decode_attn_fp16(st.cfg, 0, to_dev(q[None], "fp32"), ctx, 2049, k16, v16)
    ref16 = o.attention(q, k.astype(np.float16).astype(np.float64), v.astype(np.float16).astype(np.float64))
    assert P.rel_err(out16[0].cpu().numpy().astype(np.float64), ref16) <= 2e-3
    assert stats.code_ties <= 1e-4 * stats.codes


def test_qwen_shaped_layer_prefill_then_decode_steps():
    """Qwen2.5-3B attention shape: 16 query heads, 2 KV heads, base 1e6, bf16,
    K3V3; prefill-quantize 32768 rows in one call, then decode steps that each
    append one row and attend over the whole cache."""
    bg = bgm()
    T, steps = 32768, 4
    st = P.make_setup(2, 1, 1, 2, 8, T + 64, 192, 3, 1e6, "bf16", n_cal=2048)
    layout, cache = build(st)
    kv = [P.keys_values(st, 0, h, 0, T + steps) for h in range(2)]
    append(st, layout, cache, 0, [[(kv[h][0][:T], kv[h][1][:T]) for h in range(2)]], [0])
    rows = [P.oracle_rows(st, 0, h, kv[h][0], kv[h][1]) for h in range(2)]
    stats = P.Stats()
    for h in range(2):
        check_cache(st, cache, 0, 0, h, rows[h], T, stats, f"qwen prefill h{h}")
    log("qwen prefill ties", vars(stats))
    for s in range(steps):
        pos = T + s
        append(st, layout, cache, 0, [[(kv[h][0][pos:pos + 1], kv[h][1][pos:pos + 1]) for h in range(2)]], [pos])
        q = np.concatenate([synth.cast(synth.queries(2, 0, h, pos, 8, 1e6, step=s), "bf16") for h in range(2)])
        ctx = torch.tensor([pos + 1], dtype=torch.int32, device="cuda")
        out = bg.blockgtq_decode_attn(st.cfg, layout, 0, to_dev(q[None], "bf16"), ctx, pos + 1, cache)
        out = out[0].cpu().numpy().astype(np.float64)
        for h in range(2):
            ref = P.oracle_attention(st, 0, h, q[h * 8:(h + 1) * 8], rows[h], pos + 1)
            err = P.rel_err(out[h * 8:(h + 1) * 8], ref)
            log("qwen step", s, "head", h, "rel err", err)
            assert err <= 2e-3
    for h in range(2):
        check_cache(st, cache, 0, 0, h, rows[h], T + steps, stats, f"qwen final h{h}")
    assert stats.code_ties <= 1e-4 * stats.codes


@pytest.mark.parametrize("k_budget,v_bits", [(128, 2), (192, 3), (64, 1), (512, 8)])
def test_uniform_tq_mse_layout(k_budget, v_bits):
    """The uniform TQ-MSE K layout (every block at k_budget / 64 bits: one K
    group of all 128 coordinates, one K radius per row), bf16, a ragged batch
    of two sequences x 2 KV heads, G = 4: codes and radii bit-exact up to
    counted ties, attention within 2e-3 of the oracle for several split
    counts, a one-row and a tile-crossing context included."""
    bg = bgm()
    st = P.make_setup(5, 1, 2, 2, 4, 3072, k_budget, v_bits, 5e5, "bf16", uniform=True)
    assert (st.bits == k_budget // 64).all() and (st.bits_oracle == st.bits).all()
    layout, cache = build(st)
    lens = [3000, 1301]
    allkv = {(b, h): P.keys_values(st, 0, h, 1000 * b, lens[b]) for b in range(2) for h in range(2)}
    # one prefill call: sequence 1's rows beyond its length are other rows
    pre = [[(np.concatenate([allkv[b, h][0], allkv[0, h][0][:lens[0] - lens[b]]]),
             np.concatenate([allkv[b, h][1], allkv[0, h][1][:lens[0] - lens[b]]])) for h in range(2)]
           for b in range(2)]
    append(st, layout, cache, 0, pre, [0, 0])
    stats = P.Stats()
    rows = {}
    for b in range(2):
        for h in range(2):
            rows[b, h] = P.oracle_rows(st, 0, h, allkv[b, h][0], allkv[b, h][1])
            assert rows[b, h].knorms.shape[1] == 1
            check_cache(st, cache, 0, b, h, rows[b, h], lens[b], stats, f"uniform K{k_budget // 64} b{b} h{h}")
    log("uniform", k_budget, v_bits, "ties", vars(stats))
    q = np.stack([np.concatenate([synth.cast(synth.queries(5, b, h, 0, 4, 5e5), "bf16") for h in range(2)])
                  for b in range(2)])
    for ctxl in ([3000, 1301], [1, 65]):
        ctx = torch.tensor(ctxl, dtype=torch.int32, device="cuda")
        for ns in (0, 1, 4):
            out = bg.blockgtq_decode_attn(st.cfg, layout, 0, to_dev(q, "bf16"), ctx, max(ctxl), cache,
                                          n_splits=ns).cpu().numpy().astype(np.float64)
            for b in range(2):
                for h in range(2):
                    ref = P.oracle_attention(st, 0, h, q[b, h * 4:(h + 1) * 4], rows[b, h], ctxl[b])
                    err = P.rel_err(out[b, h * 4:(h + 1) * 4], ref)
                    assert err <= 2e-3, (k_budget, v_bits, ctxl, ns, b, h, err)
    assert stats.code_ties <= 1e-4 * stats.codes


@pytest.mark.parametrize("case", ["llama_k2v2_bf16_chunked", "qwen_k3v3_fp32", "uniform_k8v8", "uniform_k2v2"])
def test_prefill_attention_over_packed_cache(case):
    """Causal prefill attention over the packed cache (one layer per call):
    every query row attends rows 0 .. its position; a batch of two with
    different start positions (a chunked prefill after 700 cached rows), a
    query count that leaves a ragged last tile, G = 4 and 8, mixed and
    uniform K layouts, bf16 and fp32 inputs; against the oracle within 2e-3."""
    bg = bgm()
    if case == "llama_k2v2_bf16_chunked":
        st = P.make_setup(7, 2, 2, 2, 4, 1024, 128, 2, 5e5, "bf16")
        layer, pos0, n_q = 1, [0, 700], 300
    elif case == "qwen_k3v3_fp32":
        st = P.make_setup(8, 1, 1, 2, 8, 512, 192, 3, 1e6, "fp32")
        layer, pos0, n_q = 0, [64], 129
    elif case == "uniform_k8v8":
        st = P.make_setup(9, 1, 1, 1, 4, 256, 512, 8, 1e4, "bf16", uniform=True)
        layer, pos0, n_q = 0, [5], 200
    else:  # every step 2-bit: hi x hi products only
        st = P.make_setup(10, 1, 1, 2, 4, 1024, 128, 2, 5e5, "bf16", uniform=True)
        layer, pos0, n_q = 0, [0], 1000
    B, H, G = st.cfg.batch, st.cfg.n_kv_heads, st.cfg.group
    layout, cache = build(st)
    total = [p + n_q for p in pos0]
    kv = {(b, h): P.keys_values(st, layer, h, 1000 * b, total[b]) for b in range(B) for h in range(H)}
    T = max(total)
    pre = []
    for b in range(B):
        fill = [P.keys_values(st, layer, h, 5000 + 1000 * b, T - total[b]) for h in range(H)]
        pre.append([(np.concatenate([kv[b, h][0], fill[h][0]]), np.concatenate([kv[b, h][1], fill[h][1]]))
                    for h in range(H)])
    append(st, layout, cache, layer, pre, [0] * B)
    q = np.stack([np.concatenate([synth.cast(synth.queries(st.seed, 16 * layer + b, h, pos0[b] + i, G, st.base,
                                                           step=i), st.dtype)[None] for i in range(n_q)])
                  for b in range(B) for h in range(H)])
    # q: [B*H, n_q, G, 128] -> [B, n_q, H*G, 128]
    q = q.reshape(B, H, n_q, G, 128).transpose(0, 2, 1, 3, 4).reshape(B, n_q, H * G, 128)
    log("prefill", case, "n_q", n_q, "pos0", pos0)
    qp = torch.tensor(pos0, dtype=torch.int32, device="cuda")
    out = bg.blockgtq_prefill_attn(st.cfg, layout, layer, to_dev(q, st.dtype), qp, max(total) - 1, cache)
    out = out.cpu().numpy().astype(np.float64)
    worst = 0.0
    for b in range(B):
        for h in range(H):
            rows = P.oracle_rows(st, layer, h, kv[b, h][0], kv[b, h][1])
            kh = o.dequantize_keys(rows.kcodes, rows.knorms, st.bits_oracle[layer, h], st.rot_k)
            vh = o.dequantize_values(rows.vcodes, rows.vnorms, st.rot_v, st.cfg.v_bits)
            qq = q[b, :, h * G:(h + 1) * G].reshape(n_q * G, 128)
            pos = np.repeat(pos0[b] + np.arange(n_q), G)
            ref = o.prefill_attention(qq, pos, kh, vh).reshape(n_q, G, 128)
            err = P.rel_err(out[b, :, h * G:(h + 1) * G].reshape(-1, 128), ref.reshape(-1, 128))
            worst = max(worst, err)
    log("prefill", case, "max rel err", worst)
    assert worst <= 2e-3


@pytest.mark.parametrize("k_budget,v_bits,G,n_kv,n_q,pos0,dtype", [
    (64, 1, 1, 1, 70, [0], "bf16"), (96, 3, 3, 2, 131, [61, 7], "fp32"), (448, 5, 5, 1, 33, [100], "bf16"),
    (512, 8, 8, 1, 17, [64], "fp32"), (224, 7, 6, 2, 65, [1, 190], "bf16"), (320, 6, 2, 1, 129, [0], "bf16"),
    (256, 4, 7, 2, 200, [3], "fp32"), (160, 2, 8, 8, 530, [40, 0], "bf16")])
def test_prefill_attention_tile_edges(k_budget, v_bits, G, n_kv, n_q, pos0, dtype):
    """Causal prefill attention where a tile, a workgroup or a packed row ends:
    every value width, key rows of 4 to 32 words with codes up to 8 bits (looked
    up in pairs up to 6), G = 1 to 8, single-row tails, start positions on and
    off a tile, and both workgroup shapes (the last case has more than 256
    workgroups of 128 rows).  Every head at the positions around the tile and
    workgroup edges, against the oracle within 2e-3.  A coordinate within
    rounding of a decision threshold (the tie bound of compare_codes) may hold
    another code than the oracle's, which moves every logit of its token by up
    to a whole quantization step: a head is compared at the positions before its
    first such token.  At least half of a case's heads (the head, where a case
    has one) have no such token and are compared whole."""
    bg = bgm()
    total = [p + n_q for p in pos0]
    T, B = max(total), len(pos0)
    st = P.make_setup(60 + v_bits, 1, B, n_kv, G, (T + 63) // 64 * 64, k_budget, v_bits, 5e5, dtype)
    layout, cache = build(st)
    kv = {(b, h): P.keys_values(st, 0, h, 2000 * b, T) for b in range(B) for h in range(n_kv)}
    append(st, layout, cache, 0, [[kv[b, h] for h in range(n_kv)] for b in range(B)], [0] * B)
    rng = np.random.default_rng(k_budget)
    q = synth.cast(rng.standard_normal((B, n_q, n_kv * G, 128)), dtype)
    log("prefill edges", k_budget, v_bits, G, n_q, pos0)
    out = bg.blockgtq_prefill_attn(st.cfg, layout, 0, to_dev(q, dtype),
                                   torch.tensor(pos0, dtype=torch.int32, device="cuda"), T - 1, cache)
    out = out.cpu().numpy().astype(np.float64)
    worst, stats, whole = 0.0, P.Stats(), 0
    for b in range(B):
        rows_per = max(1, 128 // G)
        want = {0, 1, n_q - 1, n_q // 2} | {e + d for e in range(rows_per, n_q, 4 * rows_per) for d in (-1, 0, 1)}
        want |= {64 * m - pos0[b] + d for m in (1, 2, 5) for d in (-1, 0)}
        at_all = np.array(sorted(i for i in want if 0 <= i < n_q))
        for h in range(n_kv):
            rows = P.oracle_rows(st, 0, h, kv[b, h][0], kv[b, h][1])
            widths = P.stream_widths(st.bits[0, h])
            kcodes = P.read_fields(cache.k_codes[0, b, h, :T].cpu().numpy().view(np.uint32), widths)
            P.compare_codes(kcodes, rows.kcodes, rows.kz, widths, P.group_dims(st.bits[0, h]), stats)
            vcodes = P.read_value_codes(cache.v_codes[0, b, h].cpu().numpy().view(np.uint32), v_bits, T)
            P.compare_codes(vcodes, rows.vcodes, rows.vz, [v_bits] * 128, np.full(128, 128), stats)
            tied = np.nonzero((kcodes != rows.kcodes).any(axis=1) | (vcodes != rows.vcodes).any(axis=1))[0]
            whole += tied.size == 0
            at = at_all if tied.size == 0 else at_all[pos0[b] + at_all < tied[0]]
            if at.size == 0:
                continue
            kh = o.dequantize_keys(rows.kcodes, rows.knorms, st.bits_oracle[0, h], st.rot_k)
            vh = o.dequantize_values(rows.vcodes, rows.vnorms, st.rot_v, v_bits)
            qq = q[b, at, h * G:(h + 1) * G].reshape(-1, 128)
            ref = o.prefill_attention(qq, np.repeat(pos0[b] + at, G), kh, vh)
            worst = max(worst, P.rel_err(out[b, at, h * G:(h + 1) * G].reshape(-1, 128), ref))
    log("prefill edges max rel err", worst, "heads compared whole", whole, "of", B * n_kv)
    assert whole >= (B * n_kv + 1) // 2
    assert worst <= 2e-3


@pytest.mark.parametrize("n_q,n_kv,G,k_budget", [(37, 1, 4, 128), (1999, 8, 4, 192), (2731, 8, 4, 128),
                                                 (8209, 8, 8, 256)])
def test_prefill_query_rotation_matches_fp32_products(n_q, n_kv, G, k_budget):
    """bf16 queries on a 16-byte aligned buffer (exact bf16 products, both
    workgroup sizes and the several passes of a large call, partial last
    wave) against the same queries four bytes off (fp32 products), row by row.

    Rotated queries (the fp32 rows that the call leaves in its workspace): both
    sides sum 128 products of one orthonormal rotation row and x in fp32, in
    different orders, scaled by at most log2 e / 16 (a group has two dims or
    more).  One rounding of 2^-23 per term on either side (an MFMA may truncate)
    and the Cauchy-Schwarz bound of the sum give 2 * 128 * 2^-23 * log2 e / 16 *
    |x| per element, 2.8e-6 of |x|.

    Outputs: the logits (base 2) differ by at most ds = |difference of the
    rotated query| |k|, a weight by 2 ds ln 2 of it (numerator and sum) and one
    fp16 step, 2^-10 of it, and a row by as much of its weighted mean of |v|, at
    most the largest stored |v|.  Stored keys and values are up to a quarter
    longer than the given ones."""
    bg = bgm()
    st = P.make_setup(90, 1, 1, n_kv, G, (n_q + 63) // 64 * 64, k_budget, 2, 5e5, "bf16")
    layout, cache = build(st)
    g = torch.Generator(device="cuda").manual_seed(n_q)
    K, V = (torch.randn((1, n_q, n_kv, 128), generator=g, device="cuda").bfloat16() for _ in range(2))
    at = torch.zeros(1, dtype=torch.int32, device="cuda")
    bg.blockgtq_quantize_append(st.cfg, layout, 0, K, V, at, cache, host_write_pos=[0])
    q = torch.randn((1, n_q, n_kv * G, 128), generator=g, device="cuda").bfloat16()
    off = torch.empty(q.numel() + 2, dtype=q.dtype, device="cuda")[2:].view(q.shape)
    off.copy_(q)
    assert q.data_ptr() % 16 == 0 and off.data_ptr() % 16 == 4
    ws = [torch.empty(bg.prefill_workspace_bytes(st.cfg, n_q), dtype=torch.uint8, device="cuda") for _ in range(2)]
    a, b = (bg.blockgtq_prefill_attn(st.cfg, layout, 0, x, at, n_q - 1, cache, workspace=w)
            for x, w in zip((q, off), ws))
    ra, rb = (w[:4 * q.numel()].view(torch.float32).view(q.shape) for w in ws)
    assert bool(torch.isfinite(ra).all()) and bool(torch.isfinite(a).all())
    limit = 2 * 128 * 2.0 ** -23 * math.log2(math.e) / 16
    rot = float(((ra - rb).abs().amax(-1) / q.float().norm(dim=-1)).max())
    kmax, vmax = (1.25 * float(x.float().norm(dim=-1).max()) for x in (K, V))
    ds = float((ra - rb).norm(dim=-1).max()) * kmax
    err = float((a - b).norm(dim=-1).max()) / vmax
    log(f"query rotation n_q {n_q} n_kv {n_kv} G {G}: rotated rows {rot:.1e} of {limit:.1e}, outputs {err:.1e}, ds {ds:.1e}")
    assert rot <= limit
    assert err <= 2.0 ** -10 + 2 * ds * math.log(2)


def test_uniform_k2_decode_many_positions():
    """Decode over a uniform K2 layout (one 2-bit group holding the whole
    key), the layout where the dropped lo part of the query matters most:
    27 contexts from 1 to 989 rows, each with the query of its position,
    against the oracle within 2e-3."""
    bg = bgm()
    st = P.make_setup(10, 1, 1, 2, 4, 1024, 128, 2, 5e5, "bf16", uniform=True)
    layout, cache = build(st)
    T = 1000
    kv = [P.keys_values(st, 0, h, 0, T) for h in range(2)]
    append(st, layout, cache, 0, [[kv[h] for h in range(2)]], [0])
    rows = [P.oracle_rows(st, 0, h, kv[h][0], kv[h][1]) for h in range(2)]
    worst = 0.0
    for ctx_n in range(1, T, 37):
        q = np.concatenate([synth.cast(synth.queries(10, 0, h, ctx_n - 1, 4, 5e5, step=ctx_n), "bf16")
                            for h in range(2)])
        ctx = torch.tensor([ctx_n], dtype=torch.int32, device="cuda")
        out = bg.blockgtq_decode_attn(st.cfg, layout, 0, to_dev(q[None], "bf16"), ctx, ctx_n, cache)
        out = out[0].cpu().numpy().astype(np.float64)
        for h in range(2):
            ref = P.oracle_attention(st, 0, h, q[h * 4:(h + 1) * 4], rows[h], ctx_n)
            worst = max(worst, P.rel_err(out[h * 4:(h + 1) * 4], ref))
    log("uniform K2 decode, max rel err", worst)
    assert worst <= 2e-3


def test_ragged_batch_unaligned_appends_and_edge_lengths():
    """Batch of 4 with different lengths, appends at positions that are not
    tile-aligned (value tiles are read-modify-written), a zero-length context,
    a one-row context, and an exactly-full tile."""
    bg = bgm()
    st = P.make_setup(4, 1, 4, 2, 4, 512, 192, 2, 5e5, "bf16", n_cal=256)
    layout, cache = build(st)
    starts = [0, 37, 300, 5]
    n1, n2 = 27, 9
    p0 = max(starts)
    allkv = {(b, h): P.keys_values(st, 0, h, 1000 * b, starts[b] + n1 + n2) for b in range(4) for h in range(2)}
    junk_k, junk_v = P.keys_values(st, 0, 1, 99999, p0)
    # one prefill call for every sequence: real rows below its start, other rows beyond
    pre = [[(np.concatenate([allkv[b, h][0][:starts[b]], junk_k[starts[b]:]]),
             np.concatenate([allkv[b, h][1][:starts[b]], junk_v[starts[b]:]])) for h in range(2)] for b in range(4)]
    append(st, layout, cache, 0, pre, [0] * 4)
    pos = list(starts)
    for n in (n1, n2):
        kvb = [[(allkv[b, h][0][pos[b]:pos[b] + n], allkv[b, h][1][pos[b]:pos[b] + n]) for h in range(2)]
               for b in range(4)]
        append(st, layout, cache, 0, kvb, pos)
        pos = [p + n for p in pos]
    stats = P.Stats()
    rows = {}
    for b in range(4):
        for h in range(2):
            rows[b, h] = P.oracle_rows(st, 0, h, allkv[b, h][0], allkv[b, h][1])
            check_cache(st, cache, 0, b, h, rows[b, h], pos[b], stats, f"ragged b{b} h{h}")
    log("ragged ties", vars(stats))
    ctx_cases = [[0, 1, 32, pos[3]], pos, [pos[0], 64, 33, 1]]
    for ctxl in ctx_cases:
        q = np.stack([np.concatenate([synth.cast(synth.queries(4, b, h, 0, 4, 5e5), "bf16") for h in range(2)])
                      for b in range(4)])
        ctx = torch.tensor(ctxl, dtype=torch.int32, device="cuda")
        for ns in (0, 3):
            out = bg.blockgtq_decode_attn(st.cfg, layout, 0, to_dev(q, "bf16"), ctx, max(ctxl), cache,
                                          n_splits=ns).cpu().numpy().astype(np.float64)
            for b in range(4):
                for h in range(2):
                    got = out[b, h * 4:(h + 1) * 4]
                    if ctxl[b] == 0:
                        assert np.all(got == 0)
                        continue
                    ref = P.oracle_attention(st, 0, h, q[b, h * 4:(h + 1) * 4], rows[b, h], ctxl[b])
                    assert P.rel_err(got, ref) <= 2e-3, (ctxl, b, h)


def test_small_appends_cross_tiles_and_value_words():
    """Decode-step appends of 1 to 4 rows (the latency-oriented append
    kernel): rows that cross a 32-row value tile, 3-bit value slots that
    straddle two 32-bit words (slots 10 and 21), two layers and two
    sequences at different offsets; then a decode over the appended rows."""
    bg = bgm()
    st = P.make_setup(6, 2, 2, 2, 4, 128, 192, 3, 5e5, "bf16", n_cal=256)
    layout, cache = build(st)
    T = 70
    kv = {(l, b, h): P.keys_values(st, l, h, 1000 * b, T) for l in range(2) for b in range(2) for h in range(2)}
    z = np.zeros((7, 128), np.float32)
    for layer in range(2):
        # a 7-row append (the tiled kernel) gives sequence 1 its first rows;
        # sequence 0 gets zero rows there, overwritten by the appends below
        pre = [[(kv[layer, 1, h][0][:7], kv[layer, 1, h][1][:7]) if b else (z, z) for h in range(2)] for b in range(2)]
        append(st, layout, cache, layer, pre, [0, 0])
    sizes = [1, 2, 3, 4, 1, 4, 3, 2, 1, 4, 4, 3, 1, 2, 4, 3, 4, 1, 2, 3]
    p = [0, 7]
    for n in sizes:
        if max(p) + n > T:
            break
        for layer in range(2):
            rows = [[(kv[layer, b, h][0][p[b]:p[b] + n], kv[layer, b, h][1][p[b]:p[b] + n]) for h in range(2)]
                    for b in range(2)]
            append(st, layout, cache, layer, rows, p)
        p = [x + n for x in p]
    stats = P.Stats()
    for layer in range(2):
        for b in range(2):
            for h in range(2):
                rows = P.oracle_rows(st, layer, h, kv[layer, b, h][0][:p[b]], kv[layer, b, h][1][:p[b]])
                check_cache(st, cache, layer, b, h, rows, p[b], stats, f"small appends l{layer} b{b} h{h}")
                q = synth.cast(synth.queries(6, layer, h, 0, 4, 5e5), "bf16")
                qq = np.zeros((2, 8, 128), np.float32)
                qq[b, h * 4:(h + 1) * 4] = q
                ctx = torch.tensor(p, dtype=torch.int32, device="cuda")
                out = bg.blockgtq_decode_attn(st.cfg, layout, layer, to_dev(qq, "bf16"), ctx, max(p), cache)
                got = out.cpu().numpy().astype(np.float64)[b, h * 4:(h + 1) * 4]
                ref = P.oracle_attention(st, layer, h, q, rows, p[b])
                assert P.rel_err(got, ref) <= 2e-3, (layer, b, h)
    log("small appends ties", vars(stats))
    assert stats.code_ties <= 1e-4 * stats.codes


@pytest.mark.parametrize("k_budget,v_bits,dtype", [(64, 1, "bf16"), (160, 3, "bf16"), (192, 5, "fp32"),
                                                    (320, 8, "bf16"), (512, 7, "fp32"), (100, 4, "bf16")])
def test_prefill_append_kernels_widths_and_offsets(k_budget, v_bits, dtype):
    """The long-append encode (quantize.hip, fp32 MFMAs): appends of 5, 17,
    33, 1100 and 6 rows per call at positions that start inside value tiles
    (3 and 31), so that consecutive calls share tiles and every tile edge
    case (a call ending or starting mid-tile, a call inside one tile) occurs;
    key rows of 4 to 32 words, value widths 1-8, bf16 and fp32 inputs, two
    layers x 2 sequences x 2 KV heads.  Every code and radius of every row
    against the oracle, bit-exact up to counted ties."""
    st = P.make_setup(50 + v_bits, 2, 2, 2, 4, 1280, k_budget, v_bits, 5e5, dtype)
    layout, cache = build(st)
    sizes = [5, 17, 33, 1100, 6]
    starts = [3, 31]
    total = sum(sizes)
    kv = {(l, b, h): P.keys_values(st, l, h, 777 * b, starts[b] + total) for l in range(2) for b in range(2)
          for h in range(2)}
    junk = {(l, h): P.keys_values(st, l, h, 99999, 31) for l in range(2) for h in range(2)}
    for layer in range(2):
        # one 31-row call: real rows below each sequence's start, other rows
        # above it (overwritten by the appends that follow)
        pre = [[(np.concatenate([kv[layer, b, h][0][:starts[b]], junk[layer, h][0][starts[b]:]]),
                 np.concatenate([kv[layer, b, h][1][:starts[b]], junk[layer, h][1][starts[b]:]])) for h in range(2)]
               for b in range(2)]
        append(st, layout, cache, layer, pre, [0, 0])
    pos = list(starts)
    for n in sizes:
        for layer in range(2):
            kvb = [[(kv[layer, b, h][0][pos[b]:pos[b] + n], kv[layer, b, h][1][pos[b]:pos[b] + n]) for h in range(2)]
                   for b in range(2)]
            append(st, layout, cache, layer, kvb, pos)
        pos = [p + n for p in pos]
    stats = P.Stats()
    for (l, b, h), (k, v) in kv.items():
        n = pos[b]
        rows = P.oracle_rows(st, l, h, k[:n], v[:n])
        check_cache(st, cache, l, b, h, rows, n, stats, f"prefill kernels K{k_budget}V{v_bits} l{l} b{b} h{h}")
    log(f"prefill kernels K{k_budget} V{v_bits} {dtype}: ties {vars(stats)}")
    assert stats.code_ties <= 1e-4 * stats.codes


def test_fp16_comparator_group8_ragged_and_poisoned_tail():
    """The fp16 comparator decode (MFMA kernel) with G = 8 query heads per KV
    head, ragged contexts that end inside a tile, several splits, and NaN in
    every cache row past the context (masked scores, zeroed values)."""
    bg = bgm()
    cfg = bg.Config(n_layers=2, batch=2, n_kv_heads=2, group=8, capacity=320, k_budget=192, v_bits=3,
                    in_dtype=bg.BGTQ_BF16)
    rng = np.random.default_rng(11)
    k = rng.standard_normal((2, 2, 2, 320, 128)).astype(np.float16)
    v = rng.standard_normal((2, 2, 2, 320, 128)).astype(np.float16)
    ctxl = [261, 77]
    for b in range(2):
        k[:, b, :, ctxl[b]:] = np.nan
        v[:, b, :, ctxl[b]:] = np.nan
    q = synth.cast(rng.standard_normal((2, 2, 16, 128)), "bf16")
    k16 = torch.from_numpy(k).cuda()
    v16 = torch.from_numpy(v).cuda()
    ctx = torch.tensor(ctxl, dtype=torch.int32, device="cuda")
    for layer in (-1, 1):
        for ns in (0, 3):
            qq = q if layer < 0 else q[layer]
            out = bg.blockgtq_decode_attn_fp16(cfg, layer, to_dev(np.ascontiguousarray(qq), "bf16"), ctx, max(ctxl),
                                               k16, v16, n_splits=ns).cpu().numpy().astype(np.float64)
            for li in ([0, 1] if layer < 0 else [1]):
                for b in range(2):
                    for h in range(2):
                        got = (out[li] if layer < 0 else out)[b, h * 8:(h + 1) * 8]
                        ref = o.attention(q[li, b, h * 8:(h + 1) * 8], k[li, b, h, :ctxl[b]].astype(np.float64),
                                          v[li, b, h, :ctxl[b]].astype(np.float64))
                        assert np.all(np.isfinite(got))
                        assert P.rel_err(got, ref) <= 2e-3, (layer, ns, li, b, h)


def test_all_layers_launch_matches_per_layer_and_split_invariance():
    bg = bgm()
    st = P.make_setup(5, 3, 2, 2, 4, 1024, 128, 2, 1e4, "bf16", n_cal=128)
    layout, c1 = build(st)
    c2 = bg.Cache(st.cfg)
    T = 700
    K = np.zeros((3, 2, T, 2, 128), np.float32)
    V = np.zeros_like(K)
    for layer in range(3):
        for b in range(2):
            for h in range(2):
                K[layer, b, :, h], V[layer, b, :, h] = P.keys_values(st, layer, h, 5000 * b, T)
    wp = torch.zeros(2, dtype=torch.int32, device="cuda")
    for layer in range(3):
        bg.blockgtq_quantize_append(st.cfg, layout, layer, to_dev(K[layer], "bf16"), to_dev(V[layer], "bf16"), wp, c1)
    bg.blockgtq_quantize_append(st.cfg, layout, -1, to_dev(K, "bf16"), to_dev(V, "bf16"), wp, c2)
    for a, b in zip((c1.k_codes, c1.k_norms, c1.v_codes, c1.v_norms), (c2.k_codes, c2.k_norms, c2.v_codes, c2.v_norms)):
        assert torch.equal(a, b)
    g = np.random.default_rng(0)
    Q = synth.cast(g.standard_normal((3, 2, 8, 128)), "bf16")
    ctx = torch.tensor([T, 411], dtype=torch.int32, device="cuda")
    outs = {}
    for ns in (1, 2, 7, 22, 0):
        outs[ns] = bg.blockgtq_decode_attn(st.cfg, layout, -1, to_dev(Q, "bf16"), ctx, T, c1, n_splits=ns)
        per = torch.stack([bg.blockgtq_decode_attn(st.cfg, layout, layer, to_dev(Q[layer], "bf16"), ctx, T, c1,
                                                   n_splits=ns) for layer in range(3)])
        assert torch.equal(per, outs[ns])
    # Probabilities enter the PV product as fp16, rounded after subtracting
    # the running max of each split, so two partitions may differ by one fp16
    # rounding of every weight: at most 2^-11 relative.
    for ns in (2, 7, 22, 0):
        rel = (outs[ns] - outs[1]).abs().max() / outs[1].abs().max()
        assert rel <= 1e-3
    again = bg.blockgtq_decode_attn(st.cfg, layout, -1, to_dev(Q, "bf16"), ctx, T, c1, n_splits=7)
    assert torch.equal(again, outs[7])
    # oracle check for a few (layer, seq, head)
    for layer, b, h in ((0, 0, 0), (2, 1, 1), (1, 1, 0)):
        rows = P.oracle_rows(st, layer, h, K[layer, b, :, h], V[layer, b, :, h])
        ctxl = int(ctx[b])
        ref = P.oracle_attention(st, layer, h, Q[layer, b, h * 4:(h + 1) * 4], rows, ctxl)
        assert P.rel_err(outs[0][layer, b, h * 4:(h + 1) * 4].cpu().numpy().astype(np.float64), ref) <= 2e-3


def test_zero_rows_and_noop_calls():
    bg = bgm()
    st = P.make_setup(6, 1, 1, 1, 2, 64, 160, 4, 1e4, "fp32", n_cal=64)
    layout, cache = build(st)
    k, v = P.keys_values(st, 0, 0, 0, 40)
    k[3] = 0.0
    v[5] = 0.0
    k[7, :64] = 0.0
    k[7, 64:] = 0.0
    append(st, layout, cache, 0, [[(k, v)]], [0])
    rows = P.oracle_rows(st, 0, 0, k, v)
    stats = P.Stats()
    check_cache(st, cache, 0, 0, 0, rows, 40, stats, "zero rows")
    assert np.all(cache.v_norms[0, 0, 0, 5].cpu().numpy() == 0)
    # n_new == 0 is a no-op
    before = cache.k_codes.clone()
    bg.blockgtq_quantize_append(st.cfg, layout, 0, to_dev(np.zeros((1, 0, 1, 128)), "fp32"),
                                to_dev(np.zeros((1, 0, 1, 128)), "fp32"),
                                torch.zeros(1, dtype=torch.int32, device="cuda"), cache)
    torch.cuda.synchronize()
    assert torch.equal(before, cache.k_codes)
    q = synth.cast(synth.queries(6, 0, 0, 40, 2, 1e4), "fp32")
    ctx = torch.tensor([40], dtype=torch.int32, device="cuda")
    out = bg.blockgtq_decode_attn(st.cfg, layout, 0, to_dev(q[None], "fp32"), ctx, 40, cache)
    ref = P.oracle_attention(st, 0, 0, q, rows, 40)
    assert P.rel_err(out[0].cpu().numpy().astype(np.float64), ref) <= 2e-3


def test_out_of_range_context_lengths_give_nan():
    """A context length outside [0, max_ctx] is read on the device, so the call
    cannot reject it: that sequence's outputs are NaN (no row is dropped
    silently), in the packed decode, the no-allocation entry point and the
    fp16 comparator, while the call's other sequences match the oracle."""
    bg = bgm()
    st = P.make_setup(8, 1, 4, 1, 4, 256, 160, 2, 1e4, "fp32", n_cal=64)
    layout, cache = build(st)
    T = 200
    kvs = [[P.keys_values(st, 0, 0, 64 * b, T)] for b in range(4)]
    append(st, layout, cache, 0, kvs, [0, 0, 0, 0])
    qs = [synth.cast(synth.queries(8, 0, 0, T, 4, 1e4), "fp32") for _ in range(4)]
    q = to_dev(np.stack(qs)[:, :, :], "fp32")
    max_ctx = 130
    ctx = torch.tensor([120, max_ctx + 1, -1, max_ctx], dtype=torch.int32, device="cuda")
    k16 = torch.zeros((1, 4, 1, 256, 128), dtype=torch.float16, device="cuda")
    v16 = torch.zeros_like(k16)
    for b in range(4):
        k16[0, b, 0, :T] = torch.from_numpy(kvs[b][0][0].astype(np.float32)).half()
        v16[0, b, 0, :T] = torch.from_numpy(kvs[b][0][1].astype(np.float32)).half()
    for n_splits in (0, 1, 3):
        outs = {"packed": bg.blockgtq_decode_attn(st.cfg, layout, 0, q, ctx, max_ctx, cache, n_splits=n_splits),
                "noalloc": bg.blockgtq_decode_attn_noalloc(st.cfg, layout, 0, q, ctx, max_ctx, cache,
                                                           torch.empty(4, 4, 128, device="cuda"), n_splits=n_splits),
                "fp16": bg.blockgtq_decode_attn_fp16(st.cfg, 0, q, ctx, max_ctx, k16, v16, n_splits=n_splits)}
        torch.cuda.synchronize()
        for name, out in outs.items():
            o_ = out.cpu().numpy()
            assert np.isnan(o_[1]).all() and np.isnan(o_[2]).all(), (name, n_splits)
            assert np.isfinite(o_[0]).all() and np.isfinite(o_[3]).all(), (name, n_splits)
        for b, c in ((0, 120), (3, max_ctx)):
            rows = P.oracle_rows(st, 0, 0, kvs[b][0][0][:c], kvs[b][0][1][:c])
            ref = P.oracle_attention(st, 0, 0, qs[b], rows, c)
            assert P.rel_err(outs["packed"][b].cpu().numpy().astype(np.float64), ref) <= P.tol_attention()


def test_argument_errors_on_device():
    bg = bgm()
    st = P.make_setup(7, 1, 1, 1, 4, 64, 192, 3, 1e4, "fp32", n_cal=32)
    layout, cache = build(st)
    q = to_dev(np.zeros((1, 4, 128)), "fp32")
    ctx = torch.tensor([10], dtype=torch.int32, device="cuda")
    small = torch.empty(16, dtype=torch.uint8, device="cuda")
    with pytest.raises(bg.BlockGTQError) as e:
        bg.blockgtq_decode_attn(st.cfg, layout, 0, q, ctx, 10, cache, workspace=small)
    assert e.value.code == -4
    with pytest.raises(bg.BlockGTQError) as e:
        bg.blockgtq_decode_attn(st.cfg, layout, 0, q, ctx, 65, cache)
    assert e.value.code == -3
    with pytest.raises(bg.BlockGTQError):
        bg.blockgtq_decode_attn(st.cfg, layout, 1, q, ctx, 10, cache)
    with pytest.raises(bg.BlockGTQError):
        bad = np.array(st.bits)
        bad[0, 0, 0] += 1
        bg.Layout(st.cfg, bad, synth.flat_rot_k(st.rot_k), st.rot_v)


@pytest.mark.parametrize("G,v_bits,k_budget", [(1, 5, 192), (2, 6, 256), (3, 7, 128), (5, 5, 192), (6, 6, 160),
                                                (7, 7, 224), (3, 1, 64), (6, 4, 320), (4, 3, 128), (8, 3, 128),
                                                (2, 3, 160)])
def test_decode_query_groups_and_value_widths(G, v_bits, k_budget):
    """Decode attention (Sec. 4) for GQA groups of 1-7 query heads (a partial
    first set of four heads for G < 4; a partial second set for G = 5..7) and
    value widths 1 and 3-7, over key rows of 8, 10, 12, 16 and 20 words (the
    3-bit cases hold 1-bit key groups, which kernels of 3-bit values decode
    with the 4-code table instead of the byte table):
    2 layers x batch 2 x 2 KV heads, bf16, contexts 1300 and 77 rows,
    all-layer calls with 0, 1 and 3 splits and single-layer calls that must
    give the same bits at 1 and 3 splits.  Codes and radii
    bit-exact up to counted ties, attention within 2e-3 of the oracle, and the
    fp16 comparator on the same group within 2e-3 of the definition on fp16
    rows."""
    bg = bgm()
    lens = [1300, 77]
    st = P.make_setup(40 + G, 2, 2, 2, G, 1344, k_budget, v_bits, 5e5, "bf16")
    L, B, H = 2, 2, 2
    layout, cache = build(st)
    kv = {(l, b, h): P.keys_values(st, l, h, 5000 * b, lens[b]) for l in range(L) for b in range(B) for h in range(H)}
    for l in range(L):
        pre = [[(np.concatenate([kv[l, b, h][0], kv[l, 0, h][0][:lens[0] - lens[b]]]),
                 np.concatenate([kv[l, b, h][1], kv[l, 0, h][1][:lens[0] - lens[b]]])) for h in range(H)]
               for b in range(B)]
        append(st, layout, cache, l, pre, [0, 0])
    rows = {key: P.oracle_rows(st, key[0], key[2], *kv[key]) for key in kv}
    stats = P.Stats()
    for (l, b, h), r in rows.items():
        check_cache(st, cache, l, b, h, r, lens[b], stats, f"G{G} bv{v_bits} L{l} b{b} h{h}")
    qs = np.stack([np.stack([np.concatenate([synth.cast(synth.queries(st.seed, l, h, lens[b] - 1, G, st.base, step=b),
                                                        "bf16") for h in range(H)]) for b in range(B)])
                   for l in range(L)])                                   # [L, B, H G, 128]
    ctx = torch.tensor(lens, dtype=torch.int32, device="cuda")
    refs = {(l, b, h): P.oracle_attention(st, l, h, qs[l, b, h * G:(h + 1) * G], rows[l, b, h], lens[b])
            for (l, b, h) in rows}
    for ns in (0, 1, 3):
        out = bg.blockgtq_decode_attn(st.cfg, layout, -1, to_dev(qs, "bf16"), ctx, max(lens), cache, n_splits=ns)
        out = out.cpu().numpy().astype(np.float64)
        for (l, b, h), ref in refs.items():
            err = P.rel_err(out[l, b, h * G:(h + 1) * G], ref)
            assert err <= P.tol_attention(), (ns, l, b, h, err)
        if ns > 0:  # same split plan: the single-layer call gives the same bits
            one = bg.blockgtq_decode_attn(st.cfg, layout, 1, to_dev(qs[1], "bf16"), ctx, max(lens), cache,
                                          n_splits=ns)
            np.testing.assert_array_equal(one.cpu().numpy(), out[1].astype(np.float32))
    log(f"G {G} v_bits {v_bits} k_budget {k_budget}: attention ok, ties {vars(stats)}")
    k16 = torch.zeros((L, B, H, st.cfg.capacity, 128), dtype=torch.float16, device="cuda")
    v16 = torch.zeros_like(k16)
    for (l, b, h), (k, v) in kv.items():
        k16[l, b, h, :lens[b]] = torch.from_numpy(k.astype(np.float32)).half().cuda()
        v16[l, b, h, :lens[b]] = torch.from_numpy(v.astype(np.float32)).half().cuda()
    out16 = bg.blockgtq_decode_attn_fp16(st.cfg, -1, to_dev(qs, "bf16"), ctx, max(lens), k16, v16, n_splits=2)
    out16 = out16.cpu().numpy().astype(np.float64)
    for (l, b, h), (k, v) in kv.items():
        ref16 = o.attention(qs[l, b, h * G:(h + 1) * G], k.astype(np.float16).astype(np.float64),
                            v.astype(np.float16).astype(np.float64))
        assert P.rel_err(out16[l, b, h * G:(h + 1) * G], ref16) <= P.tol_attention()
    assert stats.code_ties <= 1e-4 * stats.codes


@pytest.fixture(scope="module")
def llama_128k():
    """Full-size step in the launch configuration bench.py times: Llama-3.1-8B
    shape (32 layers, 8 KV heads, G = 4, base 5e5, bf16, K2V2), 131072 cached
    rows, one all-layer append of row 131072 and one all-layer decode with the
    default split plan for bench.py's max_ctx.  Keeps the inputs of two whole
    layers for the oracle."""
    bg = bgm()
    T, L, H, G = 131072, 32, 8, 4
    max_ctx = T + 25                    # bench.py default: 5 warm-up + 20 timed steps
    st = P.make_setup(3, L, 1, H, G, T + 64, 128, 2, 5e5, "bf16", n_cal=2048)
    layout, cache = build(st)
    kept_layers = (5, 27)
    kept = {}
    knew = torch.empty((L, 1, 1, H, 128), dtype=torch.bfloat16, device="cuda")
    vnew = torch.empty_like(knew)
    wp0 = torch.zeros(1, dtype=torch.int32, device="cuda")
    for layer in range(L):
        sig = np.stack([st.sigma[layer, h] for h in range(H)])
        k, v = synth.torch_layer_kv(st.seed, layer, T + 1, sig, st.base)
        bg.blockgtq_quantize_append(st.cfg, layout, layer, k[None, :T].contiguous(), v[None, :T].contiguous(), wp0,
                                    cache)
        knew[layer, 0, 0] = k[T]
        vnew[layer, 0, 0] = v[T]
        if layer in kept_layers:
            kept[layer] = (k.float().cpu().numpy(), v.float().cpu().numpy())
        del k, v
    log("llama 128k: prefill done")
    q = torch.stack([synth.torch_queries(st.seed, layer, H * G, [T], st.base)[0] for layer in range(L)])[:, None]
    q = q.contiguous()
    bg.blockgtq_quantize_append(st.cfg, layout, -1, knew, vnew, torch.tensor([T], dtype=torch.int32, device="cuda"),
                                cache)
    out = bg.blockgtq_decode_attn(st.cfg, layout, -1, q, torch.tensor([T + 1], dtype=torch.int32, device="cuda"),
                                  max_ctx, cache)
    out = out.cpu().numpy().astype(np.float64)
    yield dict(st=st, cache=cache, out=out, qh=q.float().cpu().numpy(), kept=kept, T=T, H=H, G=G)
    del layout, cache


@pytest.mark.parametrize("layer", [5, 27])
def test_llama_128k_step_whole_layer(llama_128k, layer):
    """Every KV head of one layer of the 128K Llama-shaped step checked in full
    against the oracle fed the same bf16 inputs: every code and norm of its
    131073 rows and the attention of all 32 query heads of the layer."""
    d = llama_128k
    st, T, H, G = d["st"], d["T"], d["H"], d["G"]
    k_all, v_all = d["kept"][layer]
    stats = P.Stats()
    worst = 0.0
    for head in range(H):
        rows = P.oracle_rows(st, layer, head, k_all[:, head], v_all[:, head])
        check_cache(st, d["cache"], layer, 0, head, rows, T + 1, stats, f"llama L{layer} h{head}")
        ref = P.oracle_attention(st, layer, head, d["qh"][layer, 0, head * G:(head + 1) * G], rows, T + 1)
        err = P.rel_err(d["out"][layer, 0, head * G:(head + 1) * G], ref)
        worst = max(worst, err)
        assert err <= P.tol_attention(), (head, err)
    log("llama 128k layer", layer, "all heads, worst rel err", worst, "ties", vars(stats))
    assert stats.code_ties <= 1e-4 * stats.codes


@pytest.mark.parametrize("k_budget,v_bits,G", [(128, 2, 4), (192, 3, 8)])
def test_protected_window_decode(k_budget, v_bits, G):
    """Protected-buffer regime (sink 4 + recent 128 fp16 rows beside the packed
    cache, and the 63 + 1 and 0 + 0 edges): a 100-row prefill that the window
    covers (no packed rows), a 300-row chunk that overruns the recent ring, then
    single-row decode appends; all-layer and single-layer calls, one and three
    splits; against the oracle's protected attention within 2e-3, and the empty
    window bit-identical to the plain packed decode.  K2V2 with one query set of
    4 heads, and K3V3 with two sets of 8 (the 3-bit values' 12-bit table)."""
    bg = bgm()
    st = P.make_setup(11, 2, 2, 2, G, 1024, k_budget, v_bits, 5e5, "bf16")
    L, B, H = st.cfg.n_layers, st.cfg.batch, st.cfg.n_kv_heads
    layout, cache = build(st)
    windows = {(ns, nr): torch.zeros(bg.window_bytes(st.cfg, ns, nr) // 2, dtype=torch.float16, device="cuda")
               for ns, nr in [(4, 128), (63, 1), (0, 0)]}
    T_final = 403
    kv = {(l, b, h): P.keys_values(st, l, h, 1000 * b, T_final) for l in range(L) for b in range(B) for h in range(H)}
    rows = {key: P.oracle_rows(st, key[0], key[2], *kv[key]) for key in kv}
    T = 0
    worst = 0.0
    for n in (100, 300, 1, 1, 1):
        K = np.zeros((L, B, n, H, 128), np.float32)
        V = np.zeros((L, B, n, H, 128), np.float32)
        for (l, b, h), (k, v) in kv.items():
            K[l, b, :, h], V[l, b, :, h] = k[T:T + n], v[T:T + n]
        wp = torch.tensor([T] * B, dtype=torch.int32, device="cuda")
        Kd, Vd = to_dev(K, st.dtype), to_dev(V, st.dtype)
        bg.blockgtq_quantize_append(st.cfg, layout, -1, Kd, Vd, wp, cache)
        for (ns, nr), win in windows.items():
            bg.blockgtq_window_append(st.cfg, -1, Kd, Vd, wp, ns, nr, win)
        T += n
        q = np.stack([np.stack([np.concatenate([synth.cast(synth.queries(11, 16 * l + b, h, T - 1, G, 5e5, step=T),
                                                           "bf16") for h in range(H)]) for b in range(B)])
                      for l in range(L)])
        qd = to_dev(q, "bf16")
        ctx = torch.tensor([T] * B, dtype=torch.int32, device="cuda")
        for (ns, nr), win in windows.items():
            for n_splits in (0, 3):
                log("protected window", ns, nr, "T", T, "splits", n_splits)
                out = bg.blockgtq_decode_attn_protected(st.cfg, layout, -1, qd, ctx, T, cache, win, ns, nr,
                                                        n_splits=n_splits).cpu().numpy().astype(np.float64)
                if (ns, nr) == (0, 0):
                    plain = bg.blockgtq_decode_attn(st.cfg, layout, -1, qd, ctx, T, cache, n_splits=n_splits)
                    np.testing.assert_array_equal(out, plain.cpu().numpy())
                for (l, b, h), (k, v) in kv.items():
                    r = rows[l, b, h]
                    bits = st.bits_oracle[l, h]
                    kh = o.dequantize_keys(r.kcodes[:T], r.knorms[:T], bits, st.rot_k)
                    vh = o.dequantize_values(r.vcodes[:T], r.vnorms[:T], st.rot_v, st.cfg.v_bits)
                    ref = o.protected_attention(q[l, b, h * G:(h + 1) * G], kh, vh, o.fp16_round(k[:T]),
                                                o.fp16_round(v[:T]), ns, nr)
                    worst = max(worst, P.rel_err(out[l, b, h * G:(h + 1) * G], ref))
        # a single-layer call reads the same window and cache
        out1 = bg.blockgtq_decode_attn_protected(st.cfg, layout, 1, qd[1].contiguous(), ctx, T, cache,
                                                 windows[4, 128], 4, 128).cpu().numpy().astype(np.float64)
        allc = bg.blockgtq_decode_attn_protected(st.cfg, layout, -1, qd, ctx, T, cache, windows[4, 128], 4, 128)
        np.testing.assert_allclose(out1, allc[1].cpu().numpy(), rtol=0, atol=1e-6)
    log("protected window, max rel err", worst)
    assert worst <= 2e-3


def _pre_rope(x, pos, base):
    """Undo the synthetic generator's RoPE: R_(-pos) x, fp64 (test-local)."""
    return o.rope_absolute(np.asarray(x, np.float64), -float(pos), base)


def test_rope_decode_step_against_oracle():
    """Decode steps from pre-RoPE inputs (on-device RoPE; fp32 inputs, batch 2,
    2 layers, G = 4; a 300-row prefill, then three steps with sequence b at
    position 300 - 50 b + s, so that the positions and contexts of the batch
    differ): the appended codes against the oracle's quantization of its own
    RoPE of the same pre-RoPE rows (ties counted), the outputs against the
    oracle within 2e-3."""
    bg = bgm()
    base = 5e5
    st = P.make_setup(12, 2, 2, 2, 4, 512, 128, 2, base, "fp32")
    L, B, H, G = st.cfg.n_layers, st.cfg.batch, st.cfg.n_kv_heads, st.cfg.group
    layout, cache = build(st)
    T0, n_steps = 300, 3
    kv = {(l, b, h): P.keys_values(st, l, h, 1000 * b, T0 + n_steps) for l in range(L) for b in range(B)
          for h in range(H)}
    for l in range(L):
        append(st, layout, cache, l, [[(kv[l, b, h][0][:T0], kv[l, b, h][1][:T0]) for h in range(H)]
                                      for b in range(B)], [0] * B)
    # the oracle's rows: prefill rows as given, step rows re-derived from the pre-RoPE input
    krows = {key: np.array(kv[key][0][:T0 + n_steps], np.float64) for key in kv}
    stats = P.Stats()
    worst = 0.0
    ws = torch.zeros(bg.rope_step_workspace_bytes(st.cfg, T0 + n_steps), dtype=torch.uint8, device="cuda")
    for s in range(n_steps):
        pos_of = [T0 + s - 50 * b for b in range(B)]
        kpre = np.zeros((L, B, 1, H, 128), np.float32)
        vv = np.zeros((L, B, 1, H, 128), np.float32)
        qpre = np.zeros((L, B, H * G, 128), np.float32)
        qpost = np.zeros((L, B, H * G, 128), np.float64)
        for (l, b, h), (k, v) in kv.items():
            pos = pos_of[b]
            kpre[l, b, 0, h] = _pre_rope(k[pos], pos, base)
            vv[l, b, 0, h] = v[pos]
            krows[l, b, h][pos] = np.float32(o.rope_absolute(kpre[l, b, 0, h].astype(np.float64), pos, base))
            qp = synth.queries(12, 16 * l + b, h, pos, G, base, step=pos)
            qpre[l, b, h * G:(h + 1) * G] = _pre_rope(qp, pos, base)
            qpost[l, b, h * G:(h + 1) * G] = o.rope_absolute(qpre[l, b, h * G:(h + 1) * G].astype(np.float64), pos,
                                                             base)
        posd = torch.tensor(pos_of, dtype=torch.int32, device="cuda")
        log("rope step", s, "positions", pos_of)
        out = bg.blockgtq_rope_decode_step(st.cfg, layout, base, to_dev(qpre, "fp32"), to_dev(kpre, "fp32"),
                                           to_dev(vv, "fp32"), posd, T0 + n_steps, cache, workspace=ws)
        out = out.cpu().numpy().astype(np.float64)
        for (l, b, h), (k, v) in kv.items():
            pos = pos_of[b]
            rows = P.oracle_rows(st, l, h, krows[l, b, h][:pos + 1].astype(np.float32), v[:pos + 1])
            check_cache(st, cache, l, b, h, rows, pos + 1, stats, f"rope step {s} l{l} b{b} h{h}")
            ref = P.oracle_attention(st, l, h, qpost[l, b, h * G:(h + 1) * G], rows, pos + 1)
            worst = max(worst, P.rel_err(out[l, b, h * G:(h + 1) * G], ref))
    log("rope step, max rel err", worst, "stats", vars(stats))
    assert stats.code_ties <= 1e-4 * stats.codes
    assert worst <= 2e-3


def test_rope_step_graph_replay():
    """The pre-RoPE step captured once in a graph and replayed for four
    positions (new inputs and positions copied into the captured buffers
    between replays, with eager work and synchronizations in between): every
    replay's output and cache equal an eager run of the same calls on a twin
    cache, bit for bit (bf16 inputs)."""
    bg = bgm()
    base = 1e4
    st = P.make_setup(13, 2, 1, 2, 4, 256, 128, 2, base, "bf16")
    L, B, H, G = st.cfg.n_layers, st.cfg.batch, st.cfg.n_kv_heads, st.cfg.group
    layout, cache_g = build(st)
    cache_e = bg.Cache(st.cfg)
    T0 = 100
    for l in range(L):
        kvl = [[P.keys_values(st, l, h, 0, T0) for h in range(H)]]
        append(st, layout, cache_g, l, kvl, [0])
        append(st, layout, cache_e, l, kvl, [0])
    rng = np.random.default_rng(5)
    max_ctx = T0 + 4
    q_in = torch.zeros((L, B, H * G, 128), dtype=torch.bfloat16, device="cuda")
    k_in = torch.zeros((L, B, 1, H, 128), dtype=torch.bfloat16, device="cuda")
    v_in = torch.zeros_like(k_in)
    pos = torch.zeros(B, dtype=torch.int32, device="cuda")
    out_g = torch.zeros((L, B, H * G, 128), dtype=torch.float32, device="cuda")
    ws_g = torch.zeros(bg.rope_step_workspace_bytes(st.cfg, max_ctx), dtype=torch.uint8, device="cuda")
    ws_e = torch.zeros_like(ws_g)
    torch.cuda.synchronize()
    side = torch.cuda.Stream()
    graph = torch.cuda.CUDAGraph()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        with torch.cuda.graph(graph, stream=side):
            bg.blockgtq_rope_decode_step(st.cfg, layout, base, q_in, k_in, v_in, pos, max_ctx, cache_g, out=out_g,
                                         workspace=ws_g, stream=side)
    torch.cuda.synchronize()
    for s in range(4):
        q = torch.from_numpy(rng.standard_normal((L, B, H * G, 128)).astype(np.float32)).to("cuda", torch.bfloat16)
        k = torch.from_numpy(rng.standard_normal((L, B, 1, H, 128)).astype(np.float32) * 3).to("cuda", torch.bfloat16)
        v = torch.from_numpy(rng.standard_normal((L, B, 1, H, 128)).astype(np.float32)).to("cuda", torch.bfloat16)
        p = torch.tensor([T0 + s], dtype=torch.int32, device="cuda")
        q_in.copy_(q)
        k_in.copy_(k)
        v_in.copy_(v)
        pos.copy_(p)
        torch.cuda.synchronize()
        log("graph replay", s)
        graph.replay()
        torch.cuda.synchronize()
        out_e = bg.blockgtq_rope_decode_step(st.cfg, layout, base, q, k, v, p, max_ctx, cache_e, workspace=ws_e)
        torch.cuda.synchronize()
        assert torch.equal(out_g, out_e), f"replay {s}"
        for name in ("k_codes", "k_norms", "v_codes", "v_norms"):
            assert torch.equal(getattr(cache_g, name), getattr(cache_e, name)), (s, name)


@pytest.mark.parametrize("T", [262144, 524288])
def test_qwen_long_context_sampled(T):
    """Long-context Qwen2.5-3B shape at full size (36 layers, 2 KV heads,
    G = 8, base 1e6, bf16, K3V3): the context prefilled in 8192-row chunks,
    then one all-layer append and decode with the split plan for 16 decode
    steps.  Whole layers (both KV heads: two layers at 256K rows, one at 512K)
    checked in full against the oracle: every code and norm of their T + 1
    rows and the attention of their 16 query heads."""
    bg = bgm()
    L, H, G, chunk = 36, 2, 8, 8192
    max_ctx = T + 16
    st = P.make_setup(5, L, 1, H, G, T + 64, 192, 3, 1e6, "bf16", n_cal=2048)
    layout, cache = build(st)
    # whole layers: both KV heads of layers 4 and 35 at 256K, of layer 35 at 512K
    samples = [(4, 0), (4, 1), (35, 0), (35, 1)] if T <= 262144 else [(35, 0), (35, 1)]
    kept = {}
    knew = torch.empty((L, 1, 1, H, 128), dtype=torch.bfloat16, device="cuda")
    vnew = torch.empty_like(knew)
    for layer in range(L):
        sig = np.stack([st.sigma[layer, h] for h in range(H)])
        k, v = synth.torch_layer_kv(st.seed, layer, T + 1, sig, st.base)
        for c0 in range(0, T, chunk):
            bg.blockgtq_quantize_append(st.cfg, layout, layer, k[None, c0:c0 + chunk].contiguous(),
                                        v[None, c0:c0 + chunk].contiguous(),
                                        torch.tensor([c0], dtype=torch.int32, device="cuda"), cache)
        knew[layer, 0, 0] = k[T]
        vnew[layer, 0, 0] = v[T]
        for sl, sh in samples:
            if sl == layer:
                kept[sl, sh] = (k[:, sh].float().cpu().numpy(), v[:, sh].float().cpu().numpy())
        del k, v
    log("qwen long context", T, ": prefill done")
    q = torch.stack([synth.torch_queries(st.seed, layer, H * G, [T], st.base)[0] for layer in range(L)])[:, None]
    q = q.contiguous()
    bg.blockgtq_quantize_append(st.cfg, layout, -1, knew, vnew, torch.tensor([T], dtype=torch.int32, device="cuda"),
                                cache)
    out = bg.blockgtq_decode_attn(st.cfg, layout, -1, q, torch.tensor([T + 1], dtype=torch.int32, device="cuda"),
                                  max_ctx, cache)
    out = out.cpu().numpy().astype(np.float64)
    qh = q.float().cpu().numpy()
    stats = P.Stats()
    for layer, head in samples:
        k, v = kept[layer, head]
        rows = P.oracle_rows(st, layer, head, k, v)
        check_cache(st, cache, layer, 0, head, rows, T + 1, stats, f"qwen {T} L{layer} h{head}")
        ref = P.oracle_attention(st, layer, head, qh[layer, 0, head * G:(head + 1) * G], rows, T + 1)
        err = P.rel_err(out[layer, 0, head * G:(head + 1) * G], ref)
        log("qwen long context", T, "layer", layer, "head", head, "rel err", err, "ties", vars(stats))
        assert err <= P.tol_attention()
    assert stats.code_ties <= 1e-4 * stats.codes


def test_ragged_batch8_llama_shape_sampled():
    """Ragged batched decode at full size: Llama-3.1-8B attention shape (8 KV
    heads, G = 4, base 5e5, bf16, K3V2; 4 layers), batch 8 with contexts drawn
    uniformly from [4K, 64K], prefilled by 16384-row quantize_append calls,
    then one step appending one row per sequence at its own position and one
    all-layer decode.  Sampled (layer, sequence, KV head) units, the shortest
    and the longest sequence among them, checked in full against the oracle."""
    bg = bgm()
    L, B, H, G, chunk = 4, 8, 8, 4, 16384
    rng = np.random.default_rng(4)
    ctx = [int(x) for x in rng.integers(4096, 65536 + 1, size=B)]
    Tm = max(ctx)
    st = P.make_setup(4, L, B, H, G, ((Tm + 1 + 63) // 64) * 64, 192, 2, 5e5, "bf16", n_cal=2048)
    layout, cache = build(st)
    b_short, b_long = int(np.argmin(ctx)), int(np.argmax(ctx))
    samples = [(0, b_short, 5), (3, b_long, 2), (2, 3, 7)]
    kept = {}
    knew = torch.empty((L, B, 1, H, 128), dtype=torch.bfloat16, device="cuda")
    vnew = torch.empty_like(knew)
    for layer in range(L):
        sig = np.stack([st.sigma[layer, h] for h in range(H)])
        kv = [synth.torch_layer_kv(st.seed * 16 + b, layer, ctx[b] + 1, sig, st.base) for b in range(B)]
        for c0 in range(0, Tm, chunk):
            n = min(chunk, Tm - c0)
            K = torch.zeros((B, n, H, 128), dtype=torch.bfloat16, device="cuda")
            V = torch.zeros_like(K)
            for b in range(B):
                m = max(0, min(n, ctx[b] - c0))
                K[b, :m] = kv[b][0][c0:c0 + m]
                V[b, :m] = kv[b][1][c0:c0 + m]
            bg.blockgtq_quantize_append(st.cfg, layout, layer, K, V,
                                        torch.tensor([c0] * B, dtype=torch.int32, device="cuda"), cache)
        for b in range(B):
            knew[layer, b, 0] = kv[b][0][ctx[b]]
            vnew[layer, b, 0] = kv[b][1][ctx[b]]
        for sl, sb, sh in samples:
            if sl == layer:
                kept[sl, sb, sh] = (kv[sb][0][:, sh].float().cpu().numpy(), kv[sb][1][:, sh].float().cpu().numpy())
        del kv
    log("ragged batch 8, contexts", ctx, ": prefill done")
    q = torch.stack([torch.stack([synth.torch_queries(st.seed * 16 + b, layer, H * G, [ctx[b]], st.base)[0]
                                  for b in range(B)]) for layer in range(L)]).contiguous()
    wp = torch.tensor(ctx, dtype=torch.int32, device="cuda")
    bg.blockgtq_quantize_append(st.cfg, layout, -1, knew, vnew, wp, cache, host_write_pos=ctx)
    out = bg.blockgtq_decode_attn(st.cfg, layout, -1, q, wp + 1, Tm + 1, cache)
    out = out.cpu().numpy().astype(np.float64)
    qh = q.float().cpu().numpy()
    stats = P.Stats()
    for layer, b, head in samples:
        k, v = kept[layer, b, head]
        rows = P.oracle_rows(st, layer, head, k, v)
        check_cache(st, cache, layer, b, head, rows, ctx[b] + 1, stats, f"ragged L{layer} b{b} h{head}")
        ref = P.oracle_attention(st, layer, head, qh[layer, b, head * G:(head + 1) * G], rows, ctx[b] + 1)
        err = P.rel_err(out[layer, b, head * G:(head + 1) * G], ref)
        log("ragged batch 8 layer", layer, "seq", b, "ctx", ctx[b] + 1, "head", head, "rel err", err)
        assert err <= P.tol_attention()
    assert stats.code_ties <= 1e-4 * stats.codes
