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
    # one live row, 16 K per wave (d 128: one chunk for each of 8 waves), widths of a single tile pair
    small("v_f32_one", seed=120, dtype="f32", d_model=128, n_heads=2, n_kv_heads=2, ffn_dim=32, vocab=64, batch=1,
          prompt_len=3, block_size=1, n_inflight=1, gen_len=6),
    # depths that leave some waves without a chunk (80 = 5 chunks) or with uneven ones (336 = 21), 19 rows
    small("v_f32_uneven", seed=121, dtype="f32", d_model=320, n_heads=5, n_kv_heads=1, ffn_dim=352, vocab=192, batch=1,
          prompt_len=19, block_size=19, n_inflight=1, gen_len=38),
    # head_dim 128, more than 256 keys (every wave of the attention walks several key tiles, the last one partial)
    small("v_f32_keys", seed=122, dtype="f32", n_heads=4, n_kv_heads=2, head_dim=128, batch=1, prompt_len=602,
          block_size=7, n_inflight=2, gen_len=28),
    # a prefill of 1,030 rows in 64-row tiles (32 columns x 17 tiles and up), steps in 16-row tiles
    small("v_f32_large", seed=123, dtype="f32", n_heads=8, n_kv_heads=4, ffn_dim=1024, batch=5, prompt_len=206,
          block_size=2, n_inflight=3, gen_len=12),
]


@pytest.mark.parametrize("w", F32, ids=lambda w: w.name)
def test_f32_tiles_and_keys(w):
    check(w)
