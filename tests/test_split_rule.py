"""Which passes run on split rows: the library's rule alone, no GPU."""
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
    (1024, 64, False), (1024, 112, True), (1024, 531, True), (2048, 65, True)])
def test_layers_take_the_faster_path(d, M, on):
    assert layer(M, d) == on


@pytest.mark.parametrize("d,M,on", [(128, 65, False), (256, 512, False), (1024, 65, False), (1024, 256, True), (2048, 65, True)])
def test_mlp_heads_take_the_faster_path(d, M, on):
    assert layer(M, d, head=1) == on
