"""GPU parity at the edges of the kernels' dispatch rules: tile remainders,
the smallest and largest windows a variant takes, and both sides of each
rule, on small models through the C ABI.

The reference is the oracle's plain float64 definition; tolerances as in
test_gpu_parity (fp32 models: confidence 1e-4, logits 1e-3; bf16 models
5e-3 and 3e-2), far above the rounding of the sums in either order (about
1e-5 at these widths) and far below what a wrong tile, key or row gives."""
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

from tests.test_gpu_parity import TOL, run_parity, small   # noqa: E402


def check(w, **kw):
    return run_parity(w, 0.9, **kw)


F32 = [
    # The products walk the depth in 128-deep stages through a ring of three (the 64-row tile, the head) or four (the
    # 16-row tile): one stage, one live row, widths of a single tile pair
    small("v_f32_one", seed=120, dtype="f32", d_model=128, n_heads=2, n_kv_heads=2, ffn_dim=32, vocab=64, batch=1,
          prompt_len=3, block_size=1, n_inflight=1, gen_len=6),
    # three stages of which the last is partial (320 = 2 x 128 + 64, 352), 19 rows
    small("v_f32_uneven", seed=121, dtype="f32", d_model=320, n_heads=5, n_kv_heads=1, ffn_dim=352, vocab=192, batch=1,
          prompt_len=19, block_size=19, n_inflight=1, gen_len=38),
    # head_dim 128, more than 512 keys (nine and more key tiles of 64, the last one partial)
    small("v_f32_keys", seed=122, dtype="f32", n_heads=4, n_kv_heads=2, head_dim=128, batch=1, prompt_len=602,
          block_size=7, n_inflight=2, gen_len=28),
    # a prefill of 1,030 rows in 64-row tiles (32 columns x 17 tiles and up), steps in 16-row tiles; eight stages
    small("v_f32_large", seed=123, dtype="f32", n_heads=8, n_kv_heads=4, ffn_dim=1024, batch=5, prompt_len=206,
          block_size=2, n_inflight=3, gen_len=12),
    # Deeper rings.  Prefills of 1,024 and 1,280 rows whose QKV and gate/up take the 64-row tile (1,344 / 32 = 42
    # column tiles x 16 row tiles and the like, from 512 on), head and steps over the same depths, and down products
    # of the 16-row tile: 4 stages (448: the three-stage ring's longest end) and 5 (608)
    small("v_f32_d448", seed=124, dtype="f32", d_model=448, n_heads=7, n_kv_heads=7, ffn_dim=608, vocab=192, batch=4,
          prompt_len=256, block_size=8, n_inflight=1, gen_len=16),
    # 5 stages (640: one steady round and an end of two), down 6 (704)
    small("v_f32_d640", seed=125, dtype="f32", d_model=640, n_heads=10, n_kv_heads=5, ffn_dim=704, vocab=192, batch=4,
          prompt_len=256, block_size=8, n_inflight=1, gen_len=16),
    # 7 stages (832 = 6.5 x 128: a steady round and an end of four, the last partial), down 7 (864: the four-stage
    # ring's first steady round)
    small("v_f32_d832", seed=126, dtype="f32", d_model=832, n_heads=13, n_kv_heads=1, ffn_dim=864, vocab=192, batch=5,
          prompt_len=256, block_size=8, n_inflight=1, gen_len=16),
]


@pytest.mark.parametrize("w", F32, ids=lambda w: w.name)
def test_f32_tiles_and_keys(w):
    check(w)


NORM = [
    # RMSNorm widths: below and off the float4 paths (d 384: not a multiple of 256), 1280 (two partly filled float4
    # a thread), 2048 and 2304 over few rows (threads side by side) and, from 257 rows on, a wave a row (8 float4 a
    # lane, and 9 of 16); the O and down products leave split partials to fold
    small("v_norm_384", seed=130, d_model=384, n_heads=3, n_kv_heads=3, head_dim=128, ffn_dim=1024, batch=2),
    small("v_norm_1280", seed=131, d_model=1280, n_heads=4, n_kv_heads=4, head_dim=64, ffn_dim=1024, batch=2),
    small("v_norm_2048", seed=132, d_model=2048, n_heads=4, n_kv_heads=2, head_dim=128, ffn_dim=4096, batch=1,
          n_layers=1, prompt_len=16, gen_len=32),
    small("v_norm_2048w", seed=133, d_model=2048, n_heads=4, n_kv_heads=2, head_dim=128, ffn_dim=1024, batch=5,
          n_layers=1, prompt_len=96, gen_len=32),
    small("v_norm_2304w", seed=134, d_model=2304, n_heads=4, n_kv_heads=2, head_dim=128, ffn_dim=512, batch=5,
          n_layers=1, prompt_len=96, gen_len=32),
]


@pytest.mark.parametrize("w", NORM, ids=lambda w: w.name)
def test_rmsnorm_widths(w):
    check(w)


TILES = [
    # one 128-deep K of two 64-deep stages (fewer than the ring holds) and depths of 3, 4 and 5 pairs of stages
    # (every tail of the three- and four-stage rings), single live rows and row remainders
    small("v_tile_k128", seed=140, d_model=128, n_heads=2, n_kv_heads=1, head_dim=64, ffn_dim=128, vocab=256, batch=1,
          prompt_len=1, block_size=1, n_inflight=1, gen_len=4),
    small("v_tile_k384", seed=141, d_model=384, n_heads=6, n_kv_heads=3, head_dim=64, ffn_dim=640, vocab=384, batch=3,
          prompt_len=51, block_size=17, n_inflight=1, gen_len=34),
    # QKV, O and head over 65 and 129 live rows of 64- and 128-row tiles (positions off multiples of 32: the V store's
    # shorter runs), hd 64 and 128
    small("v_tile_rows", seed=142, n_heads=4, n_kv_heads=2, head_dim=128, batch=3, prompt_len=43, block_size=43,
          n_inflight=1, gen_len=86),
    # four waves a 64 x 128 tile: gate/up of 64 column tiles over a capacity of 768 rows and 360 live ones (a part tile);
    # QKV in 32 x 64 tiles over 33 and 63 live rows; K of two stages in both
    small("v_tile_4waves", seed=144, d_model=128, n_heads=2, n_kv_heads=1, head_dim=64, ffn_dim=4096, batch=9,
          prompt_len=40, block_size=40, n_inflight=1, gen_len=80, n_layers=1),
    small("v_tile_33", seed=145, n_heads=4, n_kv_heads=2, head_dim=128, batch=1, prompt_len=33, block_size=33,
          n_inflight=1, gen_len=66),
    small("v_tile_63", seed=146, d_model=128, n_heads=2, n_kv_heads=1, head_dim=64, batch=3, prompt_len=21,
          block_size=21, n_inflight=1, gen_len=42),
    small("v_tile_rows64", seed=143, n_heads=8, n_kv_heads=4, head_dim=64, batch=13, prompt_len=15, block_size=5,
          n_inflight=2, gen_len=20),
]


@pytest.mark.parametrize("w", TILES, ids=lambda w: w.name)
def test_gemm_tiles(w):
    check(w)


@pytest.mark.parametrize("wq", ["fp8", "mxfp4"])
@pytest.mark.parametrize("w", TILES[:3], ids=lambda w: w.name)
def test_gemm_tiles_quantized(w, wq):
    check(w, wq=wq)


ATTN = [
    # (2, 2): up to 64 queries a kv head (a whole wave and one query beside it: 33), one split, up to three stages of keys
    (small("v_attn_22_64", seed=150, n_heads=4, n_kv_heads=4, head_dim=64, batch=2, prompt_len=33, block_size=33,
           n_inflight=1, gen_len=66), None),
    # (2, 2) for few tiles, keys in splits of which the last holds a partial stage; 65 queries: a second tile of one
    (small("v_attn_22_128", seed=151, n_heads=5, n_kv_heads=1, head_dim=128, batch=1, prompt_len=637, block_size=13,
           n_inflight=1, gen_len=26), None),
    # (4, 1): 40 tiles of 128 queries with 4 splits (hd 64: 96 queries, one group idle; hd 128: 130, a second tile)
    (small("v_attn_41_64", seed=152, n_heads=16, n_kv_heads=4, head_dim=64, batch=10, prompt_len=648, block_size=8,
           n_inflight=3, gen_len=48), (0, 9)),
    (small("v_attn_41_128", seed=153, n_heads=10, n_kv_heads=2, head_dim=128, batch=10, prompt_len=650, block_size=13,
           n_inflight=2, gen_len=26), (0, 9)),
    # (4, 2): 144 tiles over 1,100 keys, unsplit (hd 64), and 132 (hd 128)
    (small("v_attn_42_64", seed=154, n_heads=16, n_kv_heads=16, head_dim=64, batch=9, prompt_len=1036, block_size=37,
           n_inflight=2, gen_len=74), (8,)),
    (small("v_attn_42_128", seed=155, n_heads=12, n_kv_heads=12, head_dim=128, batch=11, prompt_len=990,
           block_size=33, n_inflight=3, gen_len=99), (10,)),
    # (4, 2) with the keys in two splits: 100 tiles over 2,120 keys, 80 queries each (one group of 32 idle, one half full)
    (small("v_attn_42_split64", seed=157, n_layers=1, n_heads=20, n_kv_heads=10, head_dim=64, batch=10, prompt_len=2080,
           block_size=20, n_inflight=2, gen_len=40), (7,)),
    (small("v_attn_42_split128", seed=158, n_layers=1, n_heads=20, n_kv_heads=10, head_dim=128, batch=10,
           prompt_len=2080, block_size=20, n_inflight=2, gen_len=40), (9,)),
    # more sequences than a wave has lanes for their windows, of which the last ends last
    (small("v_attn_b67", seed=156, n_heads=4, n_kv_heads=1, head_dim=64, batch=67, prompt_len=24, block_size=24,
           n_inflight=1, gen_len=48), (0, 63, 64, 66)),
]


@pytest.mark.parametrize("w,ids", ATTN, ids=lambda x: getattr(x, "name", ""))
def test_attention_shapes(w, ids):
    check(w, seq_ids=ids)


MOE = [
    # router and dispatch: every expert chosen, two chunks a wave, one row; 20 experts of 64 lanes, 6 chunks (a multiple
    # of the ring), one row past a row tile; 64 experts, 10 chunks, assignments that end within a wave's share
    small("v_moe_e5", seed=160, ffn_dim=0, n_experts=5, top_k=5, expert_ffn=128, batch=1, prompt_len=3, block_size=1,
          n_inflight=1, gen_len=6),
    small("v_moe_e20", seed=161, d_model=768, ffn_dim=0, n_experts=20, top_k=3, expert_ffn=128, n_shared=1, batch=1,
          prompt_len=17, block_size=17, n_inflight=1, gen_len=34),
    small("v_moe_e64", seed=162, d_model=1280, ffn_dim=0, n_experts=64, top_k=8, expert_ffn=128, batch=5,
          prompt_len=105, block_size=15, n_inflight=2, gen_len=30),
]


@pytest.mark.parametrize("w", MOE, ids=lambda w: w.name)
def test_moe_router_and_dispatch(w):
    check(w)


COMMIT = [
    # the commit kernel: more masked positions than it keeps in LDS (70 x 4 x 32 = 8,960), sequences beyond a wave's
    # lanes and off the four a lane sums
    (small("v_commit_8960", seed=170, n_layers=1, d_model=128, n_heads=2, n_kv_heads=2, ffn_dim=128, vocab=256,
           batch=70, prompt_len=32, block_size=32, n_inflight=4, gen_len=256), (0, 1, 63, 64, 69)),
]


@pytest.mark.parametrize("w,ids", COMMIT, ids=lambda x: getattr(x, "name", ""))
def test_commit_many_positions(w, ids):
    check(w, seq_ids=ids)


def test_mxfp4_weight_of_more_than_4_gib_of_codes():
    """Gate/up of 135,168 x 65,536 weights, 4.1 GiB of MXFP4 codes, non-zero in
    the last 1,024 columns alone, which lie past 4 GiB: blocks read from
    anywhere else are zero or another block's.  O is zero, so that every row of
    the window is the mask token's; the weights are E2M1 values times a power of
    two (exact in the format), and float64 takes the non-zero parts.  Tolerance
    as for every bf16 model; without the product the logits are off by several
    units."""
    from paper_2609_33887_amd import bd
    from tests.test_gpu_parity import _need_gpu
    _need_gpu()
    dev = torch.device("cuda", 0)
    if torch.cuda.get_device_properties(dev).total_memory < 100 << 30:
        pytest.skip("needs 60 GiB of device memory")
    d, F, V, S, D = 65536, 67584, 128, 1024, 256
    g = torch.Generator(device=dev).manual_seed(180)
    vals = torch.tensor([0.5, 1.0, 1.5, 2.0, 3.0, 4.0, 6.0], device=dev)

    def e2m1(rows, cols):
        mag = vals[torch.randint(0, 7, (rows, cols), generator=g, device=dev)]
        sign = 1 - 2 * torch.randint(0, 2, (rows, cols), generator=g, device=dev)
        return (mag * sign * 2.0 ** -8).bfloat16()

    def normal(*shape, std=0.02):
        return torch.randn(shape, generator=g, device=dev).mul_(std).bfloat16()

    def zeros(*shape):
        return torch.zeros(shape, dtype=torch.bfloat16, device=dev)

    ones = torch.ones(d, device=dev)
    embed, head = normal(V, d), normal(V, d, std=0.001)
    gate, up, down = zeros(F, d), zeros(F, d), zeros(d, F)
    gate[:, -S:], up[:, -S:], down[:D] = e2m1(F, S), e2m1(F, S), e2m1(D, F)
    tensors = [embed, ones, normal(256, d), zeros(d, 128), ones, gate, up, down, ones, head]
    cfg = bd.bd_model_cfg(n_layers=1, d_model=d, n_heads=2, n_kv_heads=1, head_dim=64, ffn_dim=F, vocab=V, n_experts=0,
                          top_k=0, expert_ffn=0, n_shared=0, rms_eps=1e-6, rope_theta=1e4, logit_scale=20.0,
                          mask_id=V - 1, dtype=bd.BD_BF16, wq=bd.BD_WQ_MXFP4)
    stream = torch.cuda.current_stream(dev).cuda_stream
    model = bd.bd_init_model(cfg, [t.data_ptr() for t in tensors], stream)
    try:
        prompt = torch.randint(0, V - 1, (1, 16), generator=g, device=dev, dtype=torch.int32)
        state = bd.bd_prefill(model, prompt.data_ptr(), 1, 16, 16, bd.decode_cfg(0.9, 1, 16))
        try:
            logits = torch.zeros(16, V, device=dev)
            bd.bd_denoise_step(model, state, 0, 0, logits.data_ptr())
            torch.cuda.synchronize(dev)
        finally:
            bd.bd_state_free(state)
    finally:
        bd.bd_model_free(model)

    def norm(v):
        return v / torch.sqrt(v.square().mean() + 1e-6)

    x = embed[V - 1].double()
    f = norm(x)[-S:]
    act = torch.nn.functional.silu(gate[:, -S:].double() @ f) * (up[:, -S:].double() @ f)
    x[:D] += down[:D].double() @ act
    want = 20.0 * (head.double() @ norm(x))
    assert want.std() > 1.0
    assert torch.isneginf(logits[:, V - 1]).all()
    assert (logits[:, :-1].double() - want[:-1]).abs().max() <= TOL["bf16"][1]


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_lm_head_argmax_beside_nan_logits(dtype):
    """Columns of NaN (head rows of NaN; the first of every 64 among them, which a
    row's reduction starts from) leave the argmax to the other columns; the
    confidence, a sum over all of them, is NaN.  Both against the logits that the
    same step returns."""
    import numpy as np
    from bd_synth import make_prompts, make_weights
    from paper_2609_33887_amd import bd
    from tests.test_gpu_parity import _need_gpu
    _need_gpu()
    w = small("v_head_nan", seed=181, dtype=dtype, n_layers=1, batch=2, prompt_len=16, gen_len=32)
    nan = np.nonzero(np.isin(np.arange(w.vocab) % 64, [0, 2, 5, 32]))[0]
    ws = make_weights(w)
    ws[-1][nan] = 0x7FC0 if dtype == "bf16" else np.nan
    model = bd.Model(w, ws)
    st = bd.State(model, make_prompts(w), w.gen_len, 0.9, w.n_inflight, w.block_size)
    conf = torch.zeros((w.batch, w.gen_len), device=model.device)
    tok = torch.full((w.batch, w.gen_len), -1, dtype=torch.int32, device=model.device)
    logits = torch.zeros((w.batch, w.gen_len, w.vocab), device=model.device)
    st.step(conf, tok, logits)
    torch.cuda.synchronize()
    assert torch.isnan(logits[..., torch.as_tensor(nan, device=model.device)]).all() and torch.isnan(conf).all()
    assert torch.equal(tok.long(), logits.nan_to_num(nan=-float("inf"), neginf=-float("inf")).argmax(-1))
    st.close()
    model.close()


def test_f32_head_over_a_million_rows():
    """1,064,960 masked positions (256 sequences x 8 blocks of 520), 66,560 row
    tiles of the fp32 head, more than a grid's second dimension holds.  Without a
    prompt every sequence is the same, and one row's arithmetic does not depend on
    the rows beside it: each sequence's confidences are those of a state of one,
    to the last bit."""
    from bd_synth import make_weights
    from paper_2609_33887_amd import bd
    from tests.test_gpu_parity import _need_gpu
    _need_gpu()
    w = small("v_f32_rows", seed=182, dtype="f32", n_layers=1, d_model=64, n_heads=1, n_kv_heads=1, ffn_dim=64, vocab=64,
              batch=256, prompt_len=0, block_size=520, n_inflight=8, gen_len=4160)
    model = bd.Model(w, make_weights(w))
    conf = {}
    for b in (1, w.batch):
        st = bd.State(model, torch.zeros((b, 0), dtype=torch.int32), w.gen_len, 0.9, w.n_inflight, w.block_size)
        conf[b] = torch.zeros((b, w.gen_len), device=model.device)
        st.step(conf[b])
        torch.cuda.synchronize()
        st.close()
    model.close()
    assert (conf[1] > 0).all() and (conf[w.batch] == conf[1]).all()


def test_f32_weights_at_any_float():
    """fp32 weights that start at any float of a buffer (a tensor of a flat
    checkpoint, say) give what the same weights at a 256-byte boundary give."""
    from bd_synth import make_prompts, make_weights
    from paper_2609_33887_amd import bd
    from tests.test_gpu_parity import _need_gpu
    _need_gpu()
    w = small("v_f32_offset", seed=183, dtype="f32", n_layers=1, batch=2, prompt_len=16, gen_len=32)
    ws = make_weights(w)
    got = []
    for shift in (0, 1, 2, 3):
        model = bd.Model(w, ws)
        bufs = []
        for t in model.tensors:
            b = torch.zeros(t.numel() + 64, device=model.device)
            b[shift:shift + t.numel()] = t.flatten()
            bufs.append(b)
        bd.bd_model_free(model.handle)
        model.handle = bd.bd_init_model(model.cfg, [b.data_ptr() + 4 * shift for b in bufs], model.stream.cuda_stream)
        st = bd.State(model, make_prompts(w), w.gen_len, 0.9, w.n_inflight, w.block_size)
        logits = torch.zeros((w.batch, w.gen_len, w.vocab), device=model.device)
        st.step(None, None, logits)
        torch.cuda.synchronize()
        got.append(logits)
        st.close()
        model.close()
    assert all(torch.equal(got[0], g) for g in got[1:])
