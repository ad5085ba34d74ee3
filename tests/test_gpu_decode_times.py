"""The decode's upload time is that of its copies: a stream of a hundred codes
uploads 70 KB of tables (tens of microseconds at most) while the host's parse
runs over all 65536 symbols, so the upload is the shorter of the two; a time
that spans the parse is not."""
import pytest
import torch

pytestmark = pytest.mark.gpu


def test_upload_leaves_out_the_parse():
    from paper_2609_00205_amd import api
    c = torch.arange(100, dtype=torch.int32, device="cuda") % 7
    e = bytes(api.huffman_encode(c))
    parse, upload = [], []
    for _ in range(30):
        assert torch.equal(api.huffman_decode(e, 100), c)
        t = api.lossless_times()
        parse.append(t["dec_parse_ms"])
        upload.append(t["dec_upload_ms"])
    assert 0 < min(upload) < min(parse), (min(upload), min(parse))
