"""Sizes of the caller's scratch as packs grow (host only): a buffer allocated once for the longest pack has to serve every shorter
one, so no query may fall as the token count rises, and the scratch that one call of a product can use has to be what its query says."""
import pytest

from paper_2408_04275_amd import binding as mm

# (kind, dtype, hidden, heads, key/value heads, head width, feed-forward width)
SHAPES = {
    "vit": (mm.ENCODER, mm.BF16, 1024, 16, 16, 64, 4096),
    "vit_huge": (mm.ENCODER, mm.BF16, 1280, 16, 16, 80, 5120),
    "decoder_7b": (mm.DECODER, mm.BF16, 4096, 32, 32, 128, 11008),
    "decoder_grouped": (mm.DECODER, mm.BF16, 4096, 32, 8, 128, 14336),
    "decoder_72b": (mm.DECODER, mm.BF16, 8192, 64, 8, 128, 29568),
    "grouped_64_wide": (mm.DECODER, mm.BF16, 1024, 16, 2, 64, 2752),
    "seven_heads_one_group": (mm.DECODER, mm.BF16, 896, 7, 1, 128, 4864),
    "f32": (mm.DECODER, mm.F32, 256, 4, 4, 64, 688),
    "f32_encoder": (mm.ENCODER, mm.F32, 512, 8, 8, 64, 2048),
}


@pytest.mark.parametrize("name", SHAPES)
def test_layer_sizes_never_fall_as_packs_grow(name):
    desc = mm.make_desc(*SHAPES[name])
    for query in (lambda T: mm.mmtrain_layer_workspace_bytes(desc, T, 4, 1), lambda T: mm.mmtrain_layer_workspace_bytes(desc, T, 4, 0),
                  lambda T: mm.mmtrain_layer_ctx_bytes(desc, T), lambda T: mm.mmtrain_stack_workspace_bytes(desc, 3, T, 4, 1, mm.STACK_RECOMPUTE),
                  lambda T: mm.mmtrain_stack_ctx_bytes(desc, 3, T, 0), lambda T: mm.mmtrain_attn_workspace_bytes(T, 4, desc.n_heads)):
        last = query(0)
        for T in list(range(1, 6400)) + list(range(6400, 40000, 29)):
            size = query(T)
            assert size >= last, (T, size, last)
            last = size


def test_backward_workspace_holds_nothing_that_no_kernel_writes():
    # what the backward pass of a 7B-shaped decoder layer keeps: the gradients of the activations, D, three arrays of partial sums of a
    # gain gradient (1024 rows at most), and scratch for products cut along K (256 blocks of 256 x 256 at most); no bias, no column sums
    kind, dtype, H, nh, nkv, d, F = SHAPES["decoder_7b"]
    desc = mm.make_desc(*SHAPES["decoder_7b"])
    for T in (64, 1024, 3072, 6144, 8192):
        activations = 2 * T * (F + 2 * F + 2 * H + nh * d + (nh + 2 * nkv) * d)
        bound = activations + 4 * T * nh + 3 * 4 * 1024 * H + 256 * 65536 * 4 + 16 * 256
        assert mm.mmtrain_layer_workspace_bytes(desc, T, 4, 1) <= bound, T
    # an encoder layer on a short pack: six arrays of partial sums, column sums in slabs of four rows (QKV's as wider heads need them), scratch for at most eight chunks
    # of a 512 x 1024 input gradient
    desc = mm.make_desc(*SHAPES["vit"])
    T, H, F = 512, 1024, 4096
    activations = 2 * T * (2 * F + 3 * H + 3 * H)
    assert mm.mmtrain_layer_workspace_bytes(desc, T, 4, 1) <= activations + 4 * T * 16 + 6 * 4 * 512 * H + 4 * 128 * (F + 3 * H) + 24 * 256 + 8 * 4 * T * H
