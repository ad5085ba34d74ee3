"""The time model's all-global term counts the copy of a padded field.

An all-global hierarchy of a field that has to be padded copies it into its
own grid first.  That copy reads every value and writes every padded node, so
whatever the card, it takes at least those bytes at the HBM's peak of 8 TB/s;
the term beside the levels (quantizer preparation alone: about 0.01 ms) can
only reach that if the calibration saw the copy."""
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", [torch.float32, torch.float64])
def test_all_global_term_counts_the_copy(dtype):
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    from paper_2609_00205_amd import api
    model = api.model_calibrate(dtype, 17)
    es = torch.empty(0, dtype=dtype).element_size()
    copy_ms = (512 ** 3 + 513 ** 3) * es / 8e12 * 1e3
    assert api.model_predict(model, (512, 512, 512), 0, 1)["quantize"] >= copy_ms
