"""smoe_forward on at most 16 tokens that reach few of the slots (route_partial_kernel, dense_*_kernel_served).

The checks are those of test_sparse_batch.py: choices and outputs against the oracle, every output bit for bit
against the five separate calls.  The shapes are the edges of this form: one token and the last batch that takes it,
every instance of the router (up to 32, 64, 128 and 256 experts, d_model in one and in several chunks), a second
product whose four parts are of odd length (d_ff = 1696), empty (d_ff = 32) or longer than what is in flight at once
(d_ff = 4096), one and several workgroups per slot and both feature widths."""
import pytest

from paper_2308_15030_amd import binding as b
from test_sparse_batch import test_router_first as check


@pytest.mark.parametrize("E,K,d,f,T,few", [
    (64, 16, 768, 3072, 1, True), (64, 16, 768, 3072, 10, True), (64, 16, 768, 3072, 13, False), (64, 10, 768, 3072, 4, True),
    (64, 10, 768, 3072, 6, False), (8, 4, 768, 3072, 1, False), (128, 128, 768, 3072, 16, True), (128, 128, 768, 3072, 17, False)])
def test_few_tokens_have_their_own_launches(E, K, d, f, T, few):
    h = b.smoe_create(E, K, d, f, 128, b.SMOE_BF16)
    assert b.smoe_describe_ffn(h, T).startswith("dense_first_kernel_served") == few
    b.smoe_destroy(h)


#        E    K    d_model d_ff  T   spare
SHAPES = [(32, 32, 768, 3072, 1, 0), (32, 32, 768, 3072, 5, 1), (64, 64, 768, 3072, 2, 0), (64, 60, 416, 1696, 16, 1),
          (64, 64, 1024, 4096, 7, 0), (128, 100, 1056, 1696, 15, 0), (100, 100, 2080, 512, 16, 1), (256, 200, 256, 1024, 16, 0),
          (200, 200, 2048, 32, 1, 0), (256, 256, 2048, 32, 3, 0)]


@pytest.mark.gpu
@pytest.mark.parametrize("E,K,d,f,T,spare", SHAPES)
def test_few_tokens(E, K, d, f, T, spare):
    check(E, K, d, f, T, spare, True)
