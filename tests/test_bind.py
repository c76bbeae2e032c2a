"""The native marshalling (_bind.so) refuses and passes on what the ctypes binding does (no GPU needed)."""
import pytest
import torch

import paper_2506_20187_amd as L

S = L.make_shape(1, 8, 8, 128, 4096, 128, 16, torch.float32)


class Pointer:
    """Not a torch.Tensor, but with the fields the binding reads."""
    is_cuda = True

    def __init__(self, address, contiguous=True):
        self.address, self.contiguous = address, contiguous

    def is_contiguous(self):
        return self.contiguous

    def data_ptr(self):
        return self.address


def test_tensors_that_are_not_on_the_gpu_are_refused_before_the_stream_is_looked_up():
    x = torch.zeros(8)
    with pytest.raises(ValueError, match="contiguous CUDA tensor"):
        L.chunk_score(S, x, x, x, x)
    with pytest.raises(ValueError, match="contiguous CUDA tensor"):
        L.chunk_topk_select(S, x, x, x, 4, 0, x, x, x)
    with pytest.raises(ValueError, match="contiguous CUDA tensor"):
        L.chunk_score(S, Pointer(4096, contiguous=False), None, None, None, stream=0)


def test_other_objects_reach_the_library_with_their_addresses():
    # a misaligned q is refused by the library itself, a missing one as well: nothing is launched
    for q in (Pointer(4096 + 8), None):
        with pytest.raises(L.LeoamError) as e:
            L.chunk_score(S, q, Pointer(4096), Pointer(4096), Pointer(4096), stream=0)
        assert e.value.status == L.binding.E_INVALID_ARG
    with pytest.raises(L.LeoamError) as e:
        L.chunk_select_attention_decode(S, *[Pointer(4096)] * 6, 4, 0, 1.0, *[Pointer(4096)] * 5,
                                        None, stream=0)
    assert e.value.status == L.binding.E_WORKSPACE


def test_wrong_kinds_of_arguments():
    with pytest.raises(TypeError):
        L.chunk_score(3, None, None, None, None, stream=0)
    with pytest.raises((TypeError, AttributeError)):
        L.chunk_score(S, 7, None, None, None, stream=0)
    with pytest.raises((TypeError, ValueError)):
        L.sparse_chunk_attention_decode(S, *[None] * 7, "scale", None, None, None, stream=0)
