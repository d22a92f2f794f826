"""Which passes run on split rows, which narrow products on the GEMV, and how the prefill and
engine attention split their keys: the library's rules alone, no GPU."""
import pytest
import torch  # noqa: F401  (before the library is loaded: both use torch's HIP runtime)

import paper_2608_15454_amd as mbp


def layer(M, d, d_ff=None, head=0):
    return bool(mbp.lib().mbp_check_split_layer(M, d, 4 * d if d_ff is None else d_ff, head))


# passes that measured slower on split rows than on the 64 x 64 tiles (us a layer 55 to 115
# against 70 to 120), and ones that measured faster
@pytest.mark.parametrize("d,M,on", [
    (128, 128, False), (128, 1024, False), (128, 32768, True), (256, 65, False), (256, 1024, False), (256, 8192, True),
    (384, 512, False), (384, 4096, True), (512, 65, False), (512, 512, True), (768, 96, False), (768, 256, True),
    (1024, 64, False), (1024, 112, True), (1024, 531, True), (2048, 65, True),
    # widths of an odd multiple of 64, whose matrices end inside a tile
    (576, 512, False), (576, 2048, True), (960, 256, False), (960, 1024, True), (1088, 1024, True), (1600, 512, True)])
def test_layers_take_the_faster_path(d, M, on):
    assert layer(M, d) == on


@pytest.mark.parametrize("d,M,on", [(128, 65, False), (256, 512, False), (1024, 65, False), (1024, 256, True), (2048, 65, True)])
def test_mlp_heads_take_the_faster_path(d, M, on):
    assert layer(M, d, head=1) == on


# blocks (64-query tiles x heads) and keys: short chains measured slower in four groups
# (100 keys, 16 heads: 9.2 us in two, 11.1 in four), long ones faster
@pytest.mark.parametrize("blocks,max_kv,mask,groups", [
    (32, 100, 0, 2), (112, 400, 0, 2), (176, 700, 0, 4), (256, 1000, 0, 4), (64, 4096, 1, 2), (272, 1088, 0, 2),
    (3071, 4096, 0, 2), (3072, 64, 0, 1)])
def test_prefill_attention_key_groups(blocks, max_kv, mask, groups):
    assert mbp.lib().mbp_check_prefill_groups(blocks, max_kv, mask) == groups


# (weights, K, rows): float32 products of K = 128 measured slower on the GEMV from 48 rows on
@pytest.mark.parametrize("wdt,K,M,on", [
    (0, 128, 1, True), (0, 128, 32, True), (0, 128, 33, False), (0, 128, 64, False), (0, 256, 64, True),
    (1, 128, 16, True), (1, 128, 17, False), (1, 256, 16, True), (1, 256, 17, False)])
def test_narrow_products(wdt, K, M, on):
    assert bool(mbp.lib().mbp_check_gemv(wdt, M, 1024, K)) == on


# rows, cached keys, float32 keys: at two and three rows one block per (row, head) measured
# slower than split keys from two load rounds of keys on (850 keys: 272 -> 279 us a step)
@pytest.mark.parametrize("M,max_ns,f32,one", [
    (1, 448, 0, True), (1, 449, 0, False), (2, 448, 0, True), (2, 850, 0, False), (3, 449, 0, False), (4, 896, 0, True),
    (4, 897, 0, False), (16, 896, 0, True), (1, 224, 1, True), (2, 225, 1, False), (8, 448, 1, True), (8, 449, 1, False)])
def test_engine_attention_splits(M, max_ns, f32, one):
    n = mbp.lib().mbp_check_engine_splits(M, 16, max_ns, 256, f32)
    assert (n == 1) == one
