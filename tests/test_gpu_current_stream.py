"""The stream a call runs on when none is named: torch's current one, at the time of the call."""
import pytest


@pytest.mark.gpu
def test_calls_follow_the_current_stream():
    import torch
    from paper_2601_22716_amd import binding
    side, seen = torch.cuda.Stream(), []
    for _ in range(2):                                  # (the first call finds the functions, later ones use them)
        for stream in (torch.cuda.default_stream(), side):
            with torch.cuda.stream(stream):
                seen.append((binding._stream(None), torch.cuda.current_stream().cuda_stream))
    assert all(got == want for got, want in seen) and len({got for got, _ in seen}) == 2
    assert binding._stream(side) == side.cuda_stream and binding._stream(7) == 7
