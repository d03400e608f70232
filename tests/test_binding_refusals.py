"""Tensors that are not on a GPU are refused on the host before any launch."""
import pytest
import torch

from paper_2609_34650_amd import binding as saf


@pytest.mark.parametrize("device", ["cpu", "cpu:0", "meta"])
def test_tensors_without_a_stream_are_refused(device):
    V = torch.zeros(1, 1, 64, 64, device=device)
    with pytest.raises((RuntimeError, ValueError, AssertionError)):
        saf._stream(V.device)
    if device != "meta":
        lse = torch.zeros(1, 1, 64)
        with pytest.raises((RuntimeError, ValueError, AssertionError)):
            saf.saf_hybrid_attn_fwd(V, V, V, [0])
        with pytest.raises((RuntimeError, ValueError, AssertionError)):
            saf.saf_hybrid_attn_bwd(V, V, V, V, V, lse, [0])


def test_outputs_of_another_shape_are_refused():
    V = torch.zeros(1, 2, 64, 64)
    lse = torch.zeros(1, 2, 64)
    with pytest.raises(ValueError, match="O has shape"):
        saf.saf_hybrid_attn_fwd(V, V, V, [0, 0], O=V[:, :1])
    with pytest.raises(ValueError, match="LSE has shape"):
        saf.saf_hybrid_attn_fwd(V, V, V, [0, 0], LSE=lse[..., :63])
    with pytest.raises(ValueError, match="dK has shape"):
        saf.saf_hybrid_attn_bwd(V, V, V, V, V, lse, [0, 0], dK=V[..., :32])
