"""The GEMM of bf16 models over many rows (encoder, cross K/V, prompt prefill) at the edges of its row and feature tiles,
through the C ABI against the CPU oracle: every logit depends on what these passes left in the caches."""
from dataclasses import replace

import pytest

import bild_inputs as bi
import oracle
from paper_2302_07863_amd import binding as b
from tests import parity
from tests.test_gpu_parity import Rig

pytestmark = pytest.mark.gpu


def _check(cfg, bar=None):
    """`bar`: the configuration whose storage type sets the tolerance."""
    R = Rig(cfg)
    ref = oracle.bild_generate(R.req, 0.4, 1.0, 4, cfg.max_new, keep_logits=True)
    st = R.state(cfg.max_new, 4)
    st.encode(R.src)
    parity.teacher_forced(st, ref, R.n0, 0.4, 1.0, bar or cfg)


@pytest.mark.parametrize("n_src", [1, 2, 15, 16, 17, 32, 33, 63, 64, 65, 129])
@pytest.mark.parametrize("act", [bi.ACT_RELU, bi.ACT_GATED_GELU])
def test_source_lengths_around_the_row_tiles(n_src, act):
    _check(bi.toy_pair(dtype=bi.DT_BF16, act=act, truncate=True, n_src=n_src, max_new=6))


@pytest.mark.parametrize("n_src", [34, 49, 65, 131])
def test_prompt_lengths_around_the_row_tiles(n_src):
    """33 rows and more of a prompt in one pass, with rotary positions; the rows behind the last whole row tile included."""
    _check(bi.toy_pair(dtype=bi.DT_BF16, act=bi.ACT_SWIGLU, pos=bi.POS_ROPE, cross=False, tied=False, truncate=True,
                       n_src=n_src, max_new=6))


@pytest.mark.parametrize("n_src", [20, 65])
@pytest.mark.parametrize("d_ff", [32, 160, 672, 896, 1440, 1664])
def test_input_counts_around_the_steps_requested_ahead(d_ff, n_src):
    """The FFN's output projection over inputs in four slices: of one step or none, of fewer steps than are requested ahead (two to six),
    of one more, of twice as many and one more, the last slice shorter (21 and 45 tiles) or past the end (5)."""
    _check(bi.toy_pair(dtype=bi.DT_BF16, d_ff=d_ff, n_src=n_src, max_new=4))


def test_wide_layers_take_the_shared_row_tiles():
    """1100 rows of a 1024-wide model with 4096 hidden units: the launch shapes whose rows go through LDS."""
    _check(bi.toy_pair(dtype=bi.DT_BF16, d=1024, heads=16, d_head=64, d_ff=4096, vocab=300, n_large=2, n_src=1100, max_new=4,
                       logit_scale=4.0))


@pytest.mark.parametrize("small,large", [(bi.DT_BF16, bi.DT_F32), (bi.DT_F32, bi.DT_BF16)])
def test_pair_of_two_storage_types_with_a_borrowed_encoder(small, large):
    """The small model attends to the encoder output of a large model that stores another type."""
    cfg = bi.toy_pair(dtype=bi.DT_BF16, n_src=40, max_new=6)   # weights that both types hold exactly
    _check(replace(cfg, small=replace(cfg.small, dtype=small), large=replace(cfg.large, dtype=large)), bar=cfg)


@pytest.mark.parametrize("n_src,act,heads,d_ff", [(1531, bi.ACT_RELU, 8, 2048), (1441, bi.ACT_RELU, 7, 1984), (1488, bi.ACT_GATED_GELU, 8, 992)])
def test_products_cut_into_one_round(n_src, act, heads, d_ff):
    """Workgroups of 96 rows x 192 and 256 features and of 48 x 128 (the large model, twice as wide): the last rows' block nearly whole, of a
    single row, whole; the last features' block short."""
    _check(bi.toy_pair(dtype=bi.DT_BF16, act=act, truncate=True, d=512, heads=heads, d_head=64, d_ff=d_ff, n_src=n_src, max_new=4, vocab=300, n_large=1, logit_scale=4.0))


@pytest.mark.parametrize("n_src,d,heads,d_ff,takes", [(151, 2560, 20, 4096, {"qkv": (48, 128), "ffn": (48, 128)}), (343, 2560, 32, 1024, {"qkv": (96, 192)}),
                                                      (451, 4096, 32, 1024, {"qkv": (96, 256)})])
def test_prompts_cut_into_one_round(n_src, d, heads, d_ff, takes):
    """The same launch shapes with rotary positions and a gated hidden state: a row block of 6, 54 and 66 rows at the end."""
    inner, rows = heads * 128, n_src - 1  # (the prompt's last token is a pass' first row)
    for what, (n, k, gated, rotary) in {"qkv": (3 * inner, d, False, True), "out": (d, inner, False, False), "ffn": (2 * d_ff, d, True, False)}.items():
        s = b.tile_shape(n, k, rows, gated, rotary)
        if what in takes:
            assert (s["rows"], s["features"]) == takes[what], (what, s)
    _check(bi.toy_pair(dtype=bi.DT_BF16, act=bi.ACT_SWIGLU, pos=bi.POS_ROPE, cross=False, tied=False, d=d, heads=heads, d_head=128, d_ff=d_ff, n_src=n_src, max_new=3, vocab=300, n_small=1,
                       n_large=2, logit_scale=4.0))
