"""The binding's checks of images and masks (no device needed): the errors
that each wrong argument raises."""
import numpy as np
import pytest
import torch


@pytest.fixture(scope="module")
def hx():
    from paper_2503_10855_amd import hx as mod
    return mod


F32 = torch.zeros((4, 6))
U8 = torch.zeros((4, 6), dtype=torch.uint8)


@pytest.mark.parametrize("src,mask,err", [
    (np.zeros((4, 6), np.float32), U8, TypeError),
    (F32, np.zeros((4, 6), np.uint8), TypeError),
    (F32.to_sparse().to(torch.int32), U8, TypeError),
    (F32.double(), U8, TypeError),
    (F32[0], U8, TypeError),
    (F32.t(), U8, TypeError),
    (torch.zeros(()), U8, TypeError),
    (F32[None], U8, TypeError),
    (F32, U8.bool(), TypeError),
    (F32, U8.t(), TypeError),
    (F32, U8[0], TypeError),
    (F32, U8[:, :5], ValueError),
    (F32, U8, ValueError),      # host tensors
])
def test_wrong_images_are_refused_by_type(hx, src, mask, err):
    with pytest.raises(err):
        hx.image_desc(src, mask)
