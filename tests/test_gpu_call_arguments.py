"""What the Python calls hand to the library: the current stream's handle, in whatever context the
call is made, and pointers of tensors that passed the shape, type and layout check."""

import threading

import pytest
import torch

from paper_2605_14037_amd import binding

pytestmark = pytest.mark.gpu


def test_current_stream_in_every_context():
    def current():
        assert (binding._stream() or 0) == torch.cuda.current_stream().cuda_stream
        return binding._stream() or 0

    plain, side = current(), torch.cuda.Stream()
    with torch.cuda.stream(side):
        assert current() == side.cuda_stream != plain
        seen = []
        thread = threading.Thread(target=lambda: seen.append(current()))    # a thread of its own: default stream
        thread.start()
        thread.join()
        assert seen == [plain]
    assert current() == plain


@pytest.mark.parametrize("make,ok", [(lambda t: t, True), (lambda t: t.float(), False), (lambda t: t.cpu(), False),
                                     (lambda t: t.transpose(0, 1), False), (lambda t: t.transpose(0, 1).contiguous(), False),
                                     (lambda t: t.reshape(-1), False), (lambda t: t[:, :, None], False)])
def test_only_matching_tensors_pass(make, ok):
    t = make(torch.zeros(3, 5, dtype=torch.bfloat16, device="cuda"))
    if ok:
        assert binding._dev_ptr(t, torch.bfloat16, (3, 5), "t") == t.data_ptr()
    else:
        with pytest.raises(ValueError, match="need a contiguous"):
            binding._dev_ptr(t, torch.bfloat16, (3, 5), "t")


def test_strided_tensors_of_the_right_shape_are_refused():
    for t in (torch.zeros(5, 3, dtype=torch.bfloat16, device="cuda").t(), torch.zeros(3, 10, dtype=torch.bfloat16, device="cuda")[:, ::2],
              torch.zeros(6, 5, dtype=torch.bfloat16, device="cuda")[::2], torch.zeros(5, dtype=torch.bfloat16, device="cuda").expand(3, 5)):
        assert t.shape == (3, 5) and t.dtype == torch.bfloat16
        with pytest.raises(ValueError, match="need a contiguous"):
            binding._dev_ptr(t, torch.bfloat16, (3, 5), "t")
