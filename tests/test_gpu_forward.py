"""GPU parity of the decoder forward (logits) against the CPU oracle, through psd_forward."""
import numpy as np
import pytest

import oracle
import paper_2510_12966_amd as psd
from paper_2510_12966_amd import synth
from paper_2510_12966_amd.synth import ModelShape

pytestmark = pytest.mark.gpu

TOL_F32 = 1e-4    # fp32 weights, fp32 accumulate
TOL_BF16 = 3e-2   # bf16 weights and KV cache, fp32 accumulate


def _desc(shape, blob, dtype, theta):
    return psd.ModelDesc(shape.n_layers, shape.d_model, shape.n_heads, shape.n_kv_heads, shape.d_ffn, shape.vocab,
                         theta, dtype, blob)


def _ctx(shapes, blobs, dtype, theta, max_seq, flags=0, k1=4, k2=8):
    d, q, t = (_desc(s, b, dtype, theta) for s, b in zip(shapes, blobs))
    return psd.Context(d, q, t, 0.3, 0.2, k1, k2, max_seq, flags=flags)


def test_tiny_fp32_stack_logits(tiny_stack):
    cfg, d, q, t, prompt = tiny_stack
    shapes, blobs = (cfg.draft, cfg.qualifier, cfg.target), (d, q, t)
    ctx = _ctx(shapes, blobs, cfg.dtype, cfg.rope_theta, 96)
    toks = synth.tokens(5, 0, 60, cfg.target.vocab)
    for which in range(3):
        om = oracle.Model(shapes[which], blobs[which], cfg.dtype, cfg.rope_theta, 96)
        ref = om.forward(toks, 0)
        # ragged widths: 16 + 1 + 2 + 3 + 5 + 17 + 16
        pos, got = 0, []
        for w in (16, 1, 2, 3, 5, 17, 16):
            got.append(ctx.forward(which, toks[pos:pos + w], pos))
            pos += w
        got = np.concatenate(got)
        assert np.abs(got - ref).max() <= TOL_F32
        # rollback: overwrite rows 20.. with other tokens, then again with the right ones
        ctx.forward(which, (toks[20:31] + 7) % cfg.target.vocab, 20)
        again = ctx.forward(which, toks[20:31], 20)
        assert np.abs(again - ref[20:31]).max() <= TOL_F32
    ctx.close()


MINI = [  # bf16 shapes that cover head dims 64 / 128, group sizes 1..4, ragged vocabulary
    (ModelShape(2, 256, 4, 2, 352, 1000), ModelShape(3, 512, 8, 2, 704, 1000), ModelShape(2, 512, 4, 4, 1024, 1000)),
]


@pytest.mark.parametrize("scramble", [0, 0x100])
def test_bf16_logits_long_context_and_paging(scramble):
    shapes = MINI[0]
    blobs = [synth.target_weights(s, 20 + i, synth.DTYPE_BF16, sigma=0.03) for i, s in enumerate(shapes)]
    n = 300   # spans three 128-key attention splits and five KV pages
    ctx = _ctx(shapes, blobs, synth.DTYPE_BF16, 10000.0, 384, flags=scramble)
    toks = synth.tokens(6, 0, n, 1000)
    for which in range(3):
        om = oracle.Model(shapes[which], blobs[which], synth.DTYPE_BF16, 10000.0, 384)
        ref = om.forward(toks, 0)
        pos, got = 0, []
        widths = [32] * 8 + [11, 1, 1, 6, 3, 17, 5]
        assert sum(widths) == n
        for w in widths:
            got.append(ctx.forward(which, toks[pos:pos + w], pos))
            pos += w
        got = np.concatenate(got)
        err = np.abs(got - ref).max()
        assert np.abs(ref).max() > 0.5 and err <= TOL_BF16, err
    ctx.close()


def test_bf16_width_invariance_is_bit_exact():
    # the same token at the same position gives the same logits bits whatever the width of the pass
    shapes = MINI[0]
    blobs = [synth.target_weights(s, 20 + i, synth.DTYPE_BF16, sigma=0.03) for i, s in enumerate(shapes)]
    ctx = _ctx(shapes, blobs, synth.DTYPE_BF16, 10000.0, 256)
    toks = synth.tokens(8, 0, 150, 1000)
    for which in (0, 2):
        ctx.forward(which, toks[:32], 0, want_logits=False)
        for p in range(32, 128, 32):
            ctx.forward(which, toks[p:p + 32], p, want_logits=False)
        wide = ctx.forward(which, toks[128:139], 128)            # width 11
        narrow = np.concatenate([ctx.forward(which, toks[128 + i:129 + i], 128 + i) for i in range(11)])
        assert np.array_equal(wide, narrow)
        two = np.concatenate([ctx.forward(which, toks[128:130], 128), ctx.forward(which, toks[130:139], 130)])
        assert np.array_equal(wide, two)
        wide32 = ctx.forward(which, toks[118:150], 118)           # 32-wide class
        assert np.array_equal(wide32[10:21], wide)
    ctx.close()


@pytest.mark.parametrize("scramble", [0, 0x100])
def test_bf16_prompt_ingestion_in_128_token_passes_is_bit_exact(scramble):
    # a prompt ingested in 128-token passes leaves the same KV cache, bit for bit, as 32-token and ragged passes:
    # the logits of what follows are identical; and they match the oracle
    shapes = MINI[0]
    blobs = [synth.target_weights(s, 20 + i, synth.DTYPE_BF16, sigma=0.03) for i, s in enumerate(shapes)]
    n = 300
    ctx = _ctx(shapes, blobs, synth.DTYPE_BF16, 10000.0, 384, flags=scramble)
    toks = synth.tokens(9, 0, n + 7, 1000)
    for which in range(3):
        out = []
        for widths in ([128, 128, 44], [32] * 9 + [12], [128, 100, 7, 65], [1, 128, 43, 128]):
            assert sum(widths) == n
            pos = 0
            for w in widths:
                ctx.forward(which, toks[pos:pos + w], pos, want_logits=False)
                pos += w
            out.append(ctx.forward(which, toks[n:n + 7], n))
        for o in out[1:]:
            assert np.array_equal(out[0], o)
        om = oracle.Model(shapes[which], blobs[which], synth.DTYPE_BF16, 10000.0, 384)
        ref = om.forward(toks, 0)[n:]
        assert np.abs(out[0] - ref).max() <= TOL_BF16
    with pytest.raises(psd.PsdError):
        ctx.forward(0, toks[:64], 0)                      # logits only up to 32 tokens per pass
    with pytest.raises(psd.PsdError):
        ctx.forward(0, toks[:129], 0, want_logits=False)
    ctx.close()


WIDE = (ModelShape(2, 256, 4, 2, 352, 1000), ModelShape(2, 512, 8, 2, 2304, 1000), ModelShape(2, 1024, 8, 4, 2560, 1000))


def test_bf16_prompt_ingestion_in_512_token_passes_is_bit_exact():
    # passes of up to 512 tokens (several 128-column groups per launch, weights and operand shared through LDS) leave
    # the same KV cache, bit for bit, as 128-token, 32-token and ragged passes; row-tile counts that are not
    # multiples of 16, K ranges of one step, both K splits (8 and 16 ranges); and the logits match the oracle
    shapes = WIDE
    blobs = [synth.target_weights(s, 40 + i, synth.DTYPE_BF16, sigma=0.03) for i, s in enumerate(shapes)]
    n = 700
    ctx = _ctx(shapes, blobs, synth.DTYPE_BF16, 10000.0, 768)
    toks = synth.tokens(11, 0, n + 5, 1000)
    for which in (1, 2):
        out = []
        for widths in ([512, 188], [128] * 5 + [60], [32] * 21 + [28], [300, 400], [1, 511, 129, 59]):
            assert sum(widths) == n
            pos = 0
            for w in widths:
                ctx.forward(which, toks[pos:pos + w], pos, want_logits=False)
                pos += w
            out.append(ctx.forward(which, toks[n:n + 5], n))
        for o in out[1:]:
            assert np.array_equal(out[0], o)
        om = oracle.Model(shapes[which], blobs[which], synth.DTYPE_BF16, 10000.0, 768)
        ref = om.forward(toks, 0)[n:]
        assert np.abs(out[0] - ref).max() <= TOL_BF16
    with pytest.raises(psd.PsdError):
        ctx.forward(0, toks[:129], 0, want_logits=False)   # a model too small for the widest kernel stays at 128
    with pytest.raises(psd.PsdError):
        ctx.forward(2, toks[:513], 0, want_logits=False)
    ctx.close()


# one shape per tile size and K split of the wide projection kernel that the models above do not reach: 256 x 128
# workgroup tiles for q/k/v with 16 K ranges (30 K steps: ranges of one and two) and with 8 (44 steps), and for gate/up,
# each with a last row group that is not full
PANEL = (ModelShape(1, 960, 15, 15, 2848, 1000), ModelShape(1, 512, 8, 8, 6176, 1000), ModelShape(1, 1408, 11, 11, 608, 1000))


@pytest.mark.parametrize("which", [0, 1, 2])
@pytest.mark.parametrize("n", [509, 512, 385])
def test_bf16_wide_projection_tiles_are_bit_exact(which, n):
    blobs = [synth.target_weights(s, 60 + i, synth.DTYPE_BF16, sigma=0.03) for i, s in enumerate(PANEL)]
    ctx = _ctx(PANEL, blobs, synth.DTYPE_BF16, 10000.0, 576)
    toks = synth.tokens(13, 0, n + 3, 1000)
    out = []
    for step in (512, 32):
        for pos in range(0, n, step):
            ctx.forward(which, toks[pos:min(pos + step, n)], pos, want_logits=False)
        out.append(ctx.forward(which, toks[n:n + 3], n))
    ctx.close()
    assert np.array_equal(out[0], out[1])
    ref = oracle.Model(PANEL[which], blobs[which], synth.DTYPE_BF16, 10000.0, 576).forward(toks, 0)[n:]
    assert np.abs(out[0] - ref).max() <= TOL_BF16


# as many kv heads as heads, a short cache and the smallest pool that is accepted: the sums of the q/k/v projection's K quarters find
# room for some of the pass's column groups at a time only: 2 + 1 groups of 128 columns, 3 + 3 of 64, and 64 columns where 128
# would fill the device
ROOM = ((ModelShape(1, 1408, 11, 11, 608, 1000), 576, 380), (ModelShape(1, 960, 15, 15, 2848, 1000), 448, 380),
        (ModelShape(1, 4096, 32, 32, 64, 1000), 128, 121))


@pytest.mark.parametrize("which", [0, 1, 2])
def test_bf16_wide_projections_in_several_launches_are_bit_exact(which):
    import ctypes as C
    from paper_2510_12966_amd import binding as b
    shape, max_seq, n = ROOM[which]
    blob = synth.target_weights(shape, 65, synth.DTYPE_BF16, sigma=0.03)
    stub = ModelShape(1, 64, 2, 1, 64, 1000)
    small = synth.target_weights(stub, 66, synth.DTYPE_BF16, sigma=0.03)
    descs = [_desc(s, w, synth.DTYPE_BF16, 10000.0) for s, w in ((stub, small), (stub, small), (shape, blob))]
    cd = [d.c() for d in descs]
    full = b.lib().psd_pool_bytes_needed(C.byref(cd[0]), C.byref(cd[1]), C.byref(cd[2]), C.byref(b._Params(0.3, 0.2, 1.0, 1, 1, max_seq, 0, 0, 0)))

    def beyond_the_attention_partials(s, widest):   # of a q/k/v projection's sums, in 256-byte pieces
        nsplit, hd = (max_seq + 127) // 128, s.d_model // s.n_heads
        sums = 4 * (s.n_heads + 2 * s.n_kv_heads) * hd * min(widest, 128 * nsplit) * 4
        return max(0, sums - nsplit * 512 * s.n_heads * (hd + 2) * 4 + 255) // 256 * 256

    least = full - 2 * beyond_the_attention_partials(stub, 128) - beyond_the_attention_partials(shape, 512 if n > 128 else 128)
    assert least < full
    with pytest.raises(psd.PsdError):
        psd.Context(*descs, 0.3, 0.2, 1, 1, max_seq, pool_bytes=least - 1)
    toks = synth.tokens(14, 0, n + 3, 1000)
    out = []
    for pool, step in ((full, 512), (least, 512), (least, 32)):
        ctx = psd.Context(*descs, 0.3, 0.2, 1, 1, max_seq, pool_bytes=pool)
        step = min(step, 512 if n > 128 else 128)
        for pos in range(0, n, step):
            ctx.forward(2, toks[pos:min(pos + step, n)], pos, want_logits=False)
        out.append(ctx.forward(2, toks[n:n + 3], n))
        ctx.close()
    assert np.array_equal(out[0], out[1]) and np.array_equal(out[0], out[2])
    ref = oracle.Model(shape, blob, synth.DTYPE_BF16, 10000.0, max_seq).forward(toks, 0)[n:]
    assert np.abs(out[0] - ref).max() <= TOL_BF16


# head dims 32 / 64 / 128 with query groups of 4, 3 and 1: the first has enough query tiles for the one-sweep attention at any
# context in 512-token passes and changes over to a workgroup per key range beyond four ranges in 100-token ones, the others
# beyond three
SWEEP = (ModelShape(1, 1024, 32, 8, 512, 200), ModelShape(1, 384, 6, 2, 256, 200), ModelShape(1, 512, 4, 4, 512, 200))


@pytest.mark.parametrize("which", [0, 1, 2])
@pytest.mark.parametrize("n", [130, 1023, 1301])
def test_bf16_wide_attention_is_bit_exact(which, n):
    # ragged last query tile, causal tiles that end inside a key range, tokens of one tile that see different ranges
    blobs = [synth.target_weights(s, 70 + i, synth.DTYPE_BF16, sigma=0.05) for i, s in enumerate(SWEEP)]
    ctx = _ctx(SWEEP, blobs, synth.DTYPE_BF16, 10000.0, 1408, flags=0x100)
    toks = synth.tokens(17, 0, n + 3, 200)
    widest = 512 if SWEEP[which].d_model >= 512 else 128
    out = []
    for step in (widest, 100, 32):
        for pos in range(0, n, step):
            ctx.forward(which, toks[pos:min(pos + step, n)], pos, want_logits=False)
        out.append(ctx.forward(which, toks[n:n + 3], n))
    ctx.close()
    assert np.array_equal(out[0], out[1]) and np.array_equal(out[0], out[2])
    ref = oracle.Model(SWEEP[which], blobs[which], synth.DTYPE_BF16, 10000.0, 1408).forward(toks, 0)[n:]
    assert np.abs(out[0] - ref).max() <= TOL_BF16

# head dims 64 and 32 sweep with two waves per query tile that take the key ranges in turn, from the second range on: one range (one
# wave a tile), an even and an odd number of them, tiles of one workgroup that end in different ranges, a workgroup with tiles beyond the last row
@pytest.mark.parametrize("shape", [ModelShape(1, 512, 8, 8, 512, 200), ModelShape(1, 512, 16, 8, 512, 200)])
@pytest.mark.parametrize("n", [33, 128, 129, 300, 384, 509])
def test_bf16_two_wave_sweep_is_bit_exact(shape, n):
    stub = ModelShape(1, 64, 2, 1, 64, 200)
    small = synth.target_weights(stub, 85, synth.DTYPE_BF16, sigma=0.03)
    blob = synth.target_weights(shape, 86, synth.DTYPE_BF16, sigma=0.05)
    ctx = _ctx((stub, stub, shape), (small, small, blob), synth.DTYPE_BF16, 10000.0, 640, k1=1, k2=1, flags=0x100)
    toks = synth.tokens(23, 0, n + 3, 200)
    out = []
    for step in (512, 32):
        for pos in range(0, n, step):
            ctx.forward(2, toks[pos:min(pos + step, n)], pos, want_logits=False)
        out.append(ctx.forward(2, toks[n:n + 3], n))
    ctx.close()
    assert np.array_equal(out[0], out[1])
    ref = oracle.Model(shape, blob, synth.DTYPE_BF16, 10000.0, 640).forward(toks, 0)[n:]
    assert np.abs(out[0] - ref).max() <= TOL_BF16


# passes of one width over a growing context: where they stop sweeping and take a workgroup per key range (384, 256 and 128 query tiles: beyond 19,
# 6 and 4 ranges) the bits stay
@pytest.mark.parametrize("shape", [ModelShape(1, 1024, 16, 4, 512, 200), ModelShape(1, 512, 16, 4, 512, 200)])
def test_bf16_wide_attention_routes_agree_where_the_rule_changes(shape):
    stub = ModelShape(1, 64, 2, 1, 64, 200)
    small = synth.target_weights(stub, 85, synth.DTYPE_BF16, sigma=0.03)
    blob = synth.target_weights(shape, 88, synth.DTYPE_BF16, sigma=0.05)
    n = 2700
    ctx = _ctx((stub, stub, shape), (small, small, blob), synth.DTYPE_BF16, 10000.0, 2816, k1=1, k2=1, flags=0x100)
    toks = synth.tokens(27, 0, n + 3, 200)
    out = []
    for step in (32, 384, 256, 128, 512):
        for pos in range(0, n, step):
            ctx.forward(2, toks[pos:min(pos + step, n)], pos, want_logits=False)
        out.append(ctx.forward(2, toks[n:n + 3], n))
    ctx.close()
    assert np.isfinite(out[0]).all()
    for o in out[1:]:
        assert np.array_equal(o, out[0])


# more than 64 key ranges: narrow passes then merge their partials in two turns of a wave's lanes, wide ones merge range by range
MANY = (ModelShape(2, 1024, 32, 8, 512, 200), ModelShape(2, 1024, 16, 16, 512, 200), ModelShape(2, 2048, 16, 16, 512, 200))


@pytest.mark.parametrize("which", [0, 1, 2])
def test_bf16_merge_of_many_key_ranges_is_bit_exact(which):
    n, m = 8000, 8512
    blobs = [synth.target_weights(s, 80 + i, synth.DTYPE_BF16, sigma=0.03) for i, s in enumerate(MANY)]
    ctx = _ctx(MANY, blobs, synth.DTYPE_BF16, 10000.0, 8640)
    toks = synth.tokens(15, 0, m + 3, 200)
    for pos in range(0, n, 500):
        ctx.forward(which, toks[pos:pos + 500], pos, want_logits=False)
    out = []
    for step in (512, 32):
        for pos in range(n, m, step):
            ctx.forward(which, toks[pos:pos + step], pos, want_logits=False)
        out.append(ctx.forward(which, toks[m:m + 3], m))
    ctx.close()
    assert np.array_equal(out[0], out[1])


# few query tiles: passes of every width merge partials, beyond 64 ranges in two turns of a wave's lanes, and beyond 124 ranges at
# head dim 128 range by range from memory; with 16 heads the 512-token passes of the same model sweep
@pytest.mark.parametrize("shape,n", [(ModelShape(1, 512, 4, 4, 512, 200), 8300), (ModelShape(1, 512, 4, 4, 512, 200), 16100),
                                     (ModelShape(1, 2048, 16, 16, 512, 200), 16100)])
def test_bf16_merge_routes_over_many_key_ranges_are_bit_exact(shape, n):
    stub = ModelShape(1, 64, 2, 1, 64, 200)
    small = synth.target_weights(stub, 83, synth.DTYPE_BF16, sigma=0.03)
    blob = synth.target_weights(shape, 84, synth.DTYPE_BF16, sigma=0.03)
    ctx = _ctx((stub, stub, shape), (small, small, blob), synth.DTYPE_BF16, 10000.0, n + 540, k1=1, k2=1)
    toks = synth.tokens(16, 0, n + 515, 200)
    for pos in range(0, n, 500):
        ctx.forward(2, toks[pos:min(pos + 500, n)], pos, want_logits=False)
    out = []
    for step in (512, 128, 32):
        for pos in range(n, n + 512, step):
            ctx.forward(2, toks[pos:pos + step], pos, want_logits=False)
        out.append(ctx.forward(2, toks[n + 512:n + 515], n + 512))
    ctx.close()
    assert np.isfinite(out[0]).all() and np.array_equal(out[0], out[1]) and np.array_equal(out[0], out[2])


def test_fp32_attention_routes_agree():
    # up to eight key ranges one launch attends and merges, beyond that two do: the same arithmetic, so a token at the
    # change-over has the same logits whichever bucket of contexts its pass was launched for; and both match the oracle
    shape = ModelShape(2, 64, 4, 2, 96, 131)
    blobs = [synth.target_weights(shape, 80 + i, synth.DTYPE_F32, sigma=0.1) for i in range(3)]
    n = 1100
    toks = synth.tokens(19, 0, n, 131)
    ref = oracle.Model(shape, blobs[0], synth.DTYPE_F32, 10000.0, 1200).forward(toks, 0)
    got = []
    for widths in ((32,), (7,)):   # launched for the longer bucket from the first pass behind 960 tokens on: at 992 and at 966
        ctx = _ctx((shape,) * 3, blobs, synth.DTYPE_F32, 10000.0, 1200, flags=0x100)
        out, pos = [], 0
        while pos < n:
            w = min(widths[0], n - pos)
            out.append(ctx.forward(0, toks[pos:pos + w], pos))
            pos += w
        got.append(np.concatenate(out))
        ctx.close()
    assert np.array_equal(got[0], got[1])
    assert np.abs(got[0] - ref).max() <= TOL_F32


@pytest.mark.parametrize("d,h,kv,f", [(32, 2, 1, 32), (256, 4, 4, 288), (288, 9, 3, 1056), (2048, 16, 4, 1120)])
def test_fp32_projection_shapes(d, h, kv, f):
    # 16 and 64 lanes per row pair (K up to 256 and beyond), K over one LDS chunk, weights over the size where columns go one
    # group after the other, an odd vocabulary, every launch class; each column's result does not depend on the width
    shape = ModelShape(1, d, h, kv, f, 77)
    blobs = [synth.target_weights(shape, 90 + i, synth.DTYPE_F32, sigma=0.05) for i in range(3)]
    ctx = _ctx((shape,) * 3, blobs, synth.DTYPE_F32, 10000.0, 96)
    toks = synth.tokens(21, 0, 90, 77)
    ref = oracle.Model(shape, blobs[0], synth.DTYPE_F32, 10000.0, 96).forward(toks, 0)
    one = np.concatenate([ctx.forward(0, toks[i:i + 1], i) for i in range(90)])
    out, pos = [], 0
    for w in (32, 2, 4, 6, 8, 3, 12, 23):
        out.append(ctx.forward(0, toks[pos:pos + w], pos))
        pos += w
    ctx.close()
    assert pos == 90 and np.array_equal(np.concatenate(out), one)
    assert np.abs(one - ref).max() <= TOL_F32


@pytest.mark.parametrize("layers,d,h,kv,f,v", [(2, 64, 4, 2, 256, 512), (3, 128, 4, 4, 512, 131), (2, 256, 8, 1, 1024, 77), (2, 512, 4, 2, 1024, 2),
                                               (1, 288, 9, 3, 992, 33), (1, 1024, 16, 8, 1024, 513)])
def test_fp32_one_launch_passes_equal_the_chain_of_launches(layers, d, h, kv, f, v):
    # small models take a pass with logits in one launch; where its bounded wait expires (at once here, for the second context) the
    # context goes on with a launch per projection: the same bits at every launch class, context length and head dim, and where the
    # one launch is not taken (more than eight key ranges, more parts than workgroups)
    shape = ModelShape(layers, d, h, kv, f, v)
    blobs = [synth.target_weights(shape, 60 + i, synth.DTYPE_F32, sigma=0.06) for i in range(3)]
    toks = synth.tokens(23, 0, 1000, v)
    got = []
    for expire in (False, True):
        ctx = _ctx((shape,) * 3, blobs, synth.DTYPE_F32, 10000.0, 1300, flags=0x100)
        before = psd.get_accept_expiries()
        if expire:
            try:
                psd.set_accept_path(3)
                ctx.forward(0, toks[:3], 0)
            finally:
                psd.set_accept_path(0)
        assert psd.get_accept_expiries() - before == (1 if expire else 0)
        out, pos = [], 0
        for w in (1, 2, 4, 5, 8, 11, 16, 24, 32, 1, 23, 1, 1, 3):
            out.append(ctx.forward(0, toks[pos:pos + w], pos))
            pos += w
        while pos < 1000:
            w = min(1 + pos % 32, 1000 - pos)
            out.append(ctx.forward(0, toks[pos:pos + w], pos))
            pos += w
        out.append(ctx.forward(0, toks[100:117], 100))   # over rows that are there already
        got.append(np.concatenate(out))
        ctx.close()
    assert np.isfinite(got[0]).all() and np.array_equal(got[0], got[1])
    ref = oracle.Model(shape, blobs[0], synth.DTYPE_F32, 10000.0, 160).forward(toks[:160], 0)
    assert np.abs(got[0][:160] - ref).max() <= TOL_F32


@pytest.mark.parametrize("widths", [(3, 1, 1, 5, 2, 1, 4, 32, 1, 17, 8, 24, 1), (1,) * 30])
def test_fp32_tags_start_again_when_they_are_used_up(widths):
    # seven passes before the end of the tags; the slots hold tag 1, which the first pass after it waits for, with a wrong value
    shape = ModelShape(3, 64, 4, 2, 256, 300)
    blob = synth.target_weights(shape, 62, synth.DTYPE_F32, sigma=0.06)
    toks = synth.tokens(25, 0, 128, 300)
    got = []
    for flags in (0, 0x400):
        ctx = _ctx((shape,) * 3, (blob,) * 3, synth.DTYPE_F32, 10000.0, 128, flags=flags)
        before = psd.get_accept_expiries()
        out, pos = [], 0
        for w in widths:
            out.append(ctx.forward(0, toks[pos:pos + w], pos))
            pos += w
        assert psd.get_accept_expiries() == before
        got.append(np.concatenate(out))
        ctx.close()
    assert np.array_equal(got[0], got[1])


def test_fp32_passes_return_to_one_launch_after_an_expired_wait():
    # what kept one launch from being resident may be over: after a pause of 1024 passes the context tries again
    shape = ModelShape(2, 64, 4, 2, 256, 512)
    blob = synth.target_weights(shape, 61, synth.DTYPE_F32, sigma=0.06)
    ctx = _ctx((shape,) * 3, (blob,) * 3, synth.DTYPE_F32, 10000.0, 300)
    toks = synth.tokens(24, 0, 8, 512)

    def route():
        ctx.profile(True)
        out = ctx.forward(0, toks, 0)
        rows = [r["name"] for r in ctx.kernel_stats() if r["launches"]]
        ctx.profile(False)
        return out, any(r.startswith("pass_f32") for r in rows)

    ref, one = route()
    assert one
    before = psd.get_accept_expiries()
    try:
        psd.set_accept_path(3)
        first = ctx.forward(0, toks, 0)
    finally:
        psd.set_accept_path(0)
    assert psd.get_accept_expiries() - before == 1
    paused, one = route()
    assert not one
    for _ in range(1022):
        ctx.forward(0, toks[:1], 0)
    assert not route()[1]
    after, one = route()
    assert one and psd.get_accept_expiries() - before == 1
    ctx.close()
    for out in (first, paused, after):
        assert np.array_equal(out, ref)


def test_bf16_ingestion_at_page_split_and_pass_boundaries():
    # prompt lengths around the KV page (64), the attention key range (128) and the pass widths (128, 512):
    # the widest passes, 32-token passes and a ragged mix leave identical logits for the tokens that follow
    shapes = WIDE
    blobs = [synth.target_weights(s, 40 + i, synth.DTYPE_BF16, sigma=0.03) for i, s in enumerate(shapes)]
    ctx = _ctx(shapes, blobs, synth.DTYPE_BF16, 10000.0, 1100)
    toks = synth.tokens(12, 0, 1100, 1000)
    for n in (1, 31, 32, 33, 63, 64, 65, 127, 128, 129, 191, 192, 193, 255, 256, 257, 511, 512, 513, 640, 1023, 1024, 1025):
        for which in (1, 2):
            rows = []
            for chunk in (512, 32, 100):
                pos = 0
                while pos < n:
                    w = min(chunk, n - pos)
                    ctx.forward(which, toks[pos:pos + w], pos, want_logits=False)
                    pos += w
                rows.append(ctx.forward(which, toks[n:n + 3], n))
            assert np.array_equal(rows[0], rows[1]) and np.array_equal(rows[0], rows[2]), (n, which)
    ctx.close()


def test_bf16_narrow_passes_across_the_merge_switch_are_bit_exact():
    # passes of up to 4 tokens let the o projection merge the attention partials itself while the context spans at
    # most a dozen key ranges, and hand the merge to a kernel of its own beyond that: on both sides of the switch
    # their logits have the bits of 11-token passes (which always use the separate kernel), and match the oracle
    shapes = MINI[0]
    blobs = [synth.target_weights(s, 20 + i, synth.DTYPE_BF16, sigma=0.03) for i, s in enumerate(shapes)]
    n0, n1 = 1408, 1672
    ctx = _ctx(shapes, blobs, synth.DTYPE_BF16, 10000.0, 1700)
    toks = synth.tokens(13, 0, n1, 1000)
    for which in (0, 2):
        for pos in range(0, n0, 32):
            ctx.forward(which, toks[pos:pos + 32], pos, want_logits=False)
        pos, narrow, k = n0, [], 0
        while pos < n1:
            w = min((4, 1, 2, 3)[k % 4], n1 - pos)
            narrow.append(ctx.forward(which, toks[pos:pos + w], pos))
            pos += w
            k += 1
        narrow = np.concatenate(narrow)
        wide = np.concatenate([ctx.forward(which, toks[p:p + 11], p) for p in range(n0, n1, 11)])   # rolls the cache back to n0 first
        assert np.array_equal(narrow, wide)
        om = oracle.Model(shapes[which], blobs[which], synth.DTYPE_BF16, 10000.0, 1700)
        ref = om.forward(toks, 0)[n0:]
        assert np.abs(narrow - ref).max() <= TOL_BF16
    ctx.close()


def test_bf16_context_length_switches_are_bit_exact():
    # the launch shape depends on how far the context reaches (who merges the attention partials past 12 key ranges,
    # four query tiles per attention workgroup past 16): the same token at the same position has the same logits
    # bits when it is computed just before and just after each switch
    shapes = MINI[0]
    blobs = [synth.target_weights(s, 20 + i, synth.DTYPE_BF16, sigma=0.03) for i, s in enumerate(shapes)]
    ctx = _ctx(shapes, blobs, synth.DTYPE_BF16, 10000.0, 2100)
    toks = synth.tokens(14, 0, 2100, 1000)
    for which in (0, 2):
        pos = 0
        for edge, w in ((12 * 128, 4), (16 * 128, 11)):
            a = edge - 64 - w + 2            # a pass of w tokens from here is bounded by edge - 2 + ... : before the switch
            while pos < a:
                n = min(32, a - pos)
                ctx.forward(which, toks[pos:pos + n], pos, want_logits=False)
                pos += n
            before = ctx.forward(which, toks[a:a + w], a)                 # context bound a + 64 <= edge
            ctx.forward(which, toks[a:a + w - 1], a, want_logits=False)   # rolls back, keeps w - 1 of them
            after = ctx.forward(which, toks[a + w - 1:a + 2 * w - 1], a + w - 1)   # bound a + w - 1 + 64 > edge
            assert np.array_equal(before[w - 1], after[0]), (which, edge)
            pos = a + 2 * w - 1
    ctx.close()


def test_bf16_narrow_passes_with_long_k_ranges_are_bit_exact():
    # passes of up to 4 tokens read the operand of a down projection with long K ranges (here 12 and 13 K steps per
    # wave, odd and even, and a ragged split of K over the waves) and of every LM head from LDS instead of registers:
    # same bits as 5- and 11-token passes, which never do, and the logits match the oracle
    shapes = (ModelShape(2, 256, 4, 2, 6144, 1000), ModelShape(1, 512, 4, 4, 6560, 1000), ModelShape(1, 256, 4, 1, 6656, 1000))
    blobs = [synth.target_weights(s, 60 + i, synth.DTYPE_BF16, sigma=0.02) for i, s in enumerate(shapes)]
    ctx = _ctx(shapes, blobs, synth.DTYPE_BF16, 10000.0, 160)
    toks = synth.tokens(15, 0, 150, 1000)
    for which in range(3):
        pos, narrow, k = 0, [], 0
        while pos < 132:
            w = min((1, 4, 2, 3)[k % 4], 132 - pos)
            narrow.append(ctx.forward(which, toks[pos:pos + w], pos))
            pos += w
            k += 1
        narrow = np.concatenate(narrow)
        wide = np.concatenate([ctx.forward(which, toks[p:p + 11], p) for p in range(0, 132, 11)])
        five = np.concatenate([ctx.forward(which, toks[p:p + 5], p) for p in range(0, 130, 5)])
        assert np.array_equal(narrow, wide) and np.array_equal(narrow[:130], five)
        om = oracle.Model(shapes[which], blobs[which], synth.DTYPE_BF16, 10000.0, 160)
        assert np.abs(narrow - om.forward(toks[:132], 0)).max() <= TOL_BF16
    ctx.close()


def test_bf16_full_size_projection_variants_are_bit_exact():
    # one-layer stacks with the draft's, the qualifier's and the target's projection shapes (small vocabulary): these are the
    # shapes that select the per-shape GEMM variants (a wave's whole K range in one round of loads for the draft's q/k/v and
    # the qualifier's o projection, the windowed four-tile gate/up kernel, the seven-tile one): passes of 1, 5 and 11 tokens
    # take them, 20-token passes take the two-column-tile kernels, and all four give the same bits; the logits match the oracle
    shapes = (ModelShape(1, 2048, 32, 8, 8192, 512), ModelShape(1, 3072, 24, 8, 8192, 512), ModelShape(1, 4096, 32, 8, 14336, 512))
    blobs = [synth.target_weights(s, 70 + i, synth.DTYPE_BF16, sigma=0.02) for i, s in enumerate(shapes)]
    ctx = _ctx(shapes, blobs, synth.DTYPE_BF16, 500000.0, 128)
    toks = synth.tokens(16, 0, 60, 512)
    for which in range(3):
        runs = []
        for w in (1, 5, 11, 20):
            runs.append(np.concatenate([ctx.forward(which, toks[p:p + w], p) for p in range(0, 55 if w != 20 else 60, w)])[:55])
        for r in runs[1:]:
            assert np.array_equal(runs[0], r), which
        om = oracle.Model(shapes[which], blobs[which], synth.DTYPE_BF16, 500000.0, 128)
        assert np.abs(runs[0] - om.forward(toks[:55], 0)).max() <= TOL_BF16
    ctx.close()


def test_small_config_target_logits_sampled():
    """Config "small" shapes (bf16, vocab 32000): one teacher-forced 24-token pass per model against the oracle."""
    cfg = synth.CONFIGS["small"]
    d, q, t, prompt = synth.build_stack(cfg)
    shapes, blobs = (cfg.draft, cfg.qualifier, cfg.target), (d, q, t)
    ctx = _ctx(shapes, blobs, cfg.dtype, cfg.rope_theta, 64)
    toks = prompt[:24]
    for which in range(3):
        om = oracle.Model(shapes[which], blobs[which], cfg.dtype, cfg.rope_theta, 32)
        ref = om.forward(toks, 0)
        got = np.concatenate([ctx.forward(which, toks[:13], 0), ctx.forward(which, toks[13:24], 13)])
        err = np.abs(got - ref).max()
        print(f"model {which}: max |logit err| = {err:.3e}, logit std = {ref.std():.3f}", flush=True)
        assert err <= TOL_BF16
    ctx.close()


def test_full_width_layer_at_the_long_context_matches_the_oracle():
    """One layer of the 8B shape (d 4096, 32 query / 8 KV heads of 128) over a context of 4.2 K tokens, the context of the
    long-prompt configuration (33 key ranges, the 48-range launch bucket): logits of a 1-token, an 11-token and a
    17-token pass against the oracle's forward over the same 4229 tokens."""
    shape = ModelShape(1, 4096, 32, 8, 512, 512)
    blob = synth.target_weights(shape, 41, synth.DTYPE_BF16, sigma=0.02)
    n0, widths = 4200, (1, 11, 17)
    n = n0 + sum(widths)
    ms = n + 3
    toks = synth.tokens(43, 0, n, shape.vocab)
    ctx = _ctx((shape,) * 3, (blob,) * 3, synth.DTYPE_BF16, 500000.0, ms, k1=5, k2=16)
    pos = 0
    while pos < n0:
        w = min(512, n0 - pos)
        ctx.forward(2, toks[pos:pos + w], pos, want_logits=False)
        pos += w
    got = []
    for w in widths:
        got.append(ctx.forward(2, toks[pos:pos + w], pos))
        pos += w
    got = np.concatenate(got)
    ctx.close()
    om = oracle.Model(shape, blob, synth.DTYPE_BF16, 500000.0, ms)
    om.forward(toks[:n0], 0, want_logits=False)
    ref = om.forward(toks[n0:], n0)
    err = float(np.abs(got - ref).max())
    print(f"full-width layer at {n0} tokens of context: max |logit err| {err:.3e}, logit std {ref.std():.3f}", flush=True)
    assert ref.std() > 0.05          # the comparison is not between two flat rows
    assert err <= TOL_BF16


def test_forward_argument_errors(tiny_stack):
    cfg, d, q, t, prompt = tiny_stack
    ctx = _ctx((cfg.draft, cfg.qualifier, cfg.target), (d, q, t), cfg.dtype, cfg.rope_theta, 48)
    with pytest.raises(psd.PsdError):
        ctx.forward(0, [cfg.target.vocab], 0)            # token out of range
    with pytest.raises(psd.PsdError):
        ctx.forward(0, [1, 2], 5)                        # gap in the cache
    with pytest.raises(psd.PsdError):
        ctx.forward(0, np.zeros(33, np.int32), 0)        # too wide
    with pytest.raises(psd.PsdError):
        ctx.forward(3, [1], 0)
    ctx.forward(0, np.zeros(32, np.int32), 0, want_logits=False)
    with pytest.raises(psd.PsdError):
        ctx.forward(0, np.zeros(32, np.int32), 32)       # past max_seq
    ctx.close()
    bad = psd.ModelDesc(2, 64, 4, 2, 256, 100, 10000.0, psd.F32, d)   # vocab differs from the others
    with pytest.raises(psd.PsdError):
        psd.Context(bad, _desc(cfg.qualifier, q, cfg.dtype, 1e4), _desc(cfg.target, t, cfg.dtype, 1e4), 0.1, 0.1, 4, 8, 64)
