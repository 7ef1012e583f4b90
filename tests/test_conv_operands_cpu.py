"""conv3x3 refuses operands that do not go together before anything is
launched: the kernels would read past the smaller one (or host memory)."""
import pytest


@pytest.mark.parametrize("shapes", [((2, 5, 9, 9), (6, 4, 3, 3), (6,)), ((2, 24, 9, 9), (6, 16, 3, 3), (6,)),
                                    ((2, 5, 9, 9), (6, 5, 1, 1), (6,)), ((2, 5, 9, 9), (6, 5, 3, 3), (5,)),
                                    ((5, 9, 9), (6, 5, 3, 3), (6,)), ((2, 5, 9, 9), (6, 5, 9), (6,)),
                                    ((2, 5, 9, 9), (6, 5, 3, 3), (6,))])
def test_refused(shapes, monkeypatch):
    import torch
    from paper_1608_05238_amd import denoise as D
    monkeypatch.setattr(D.L, "load", lambda: pytest.fail("reached the library"))
    monkeypatch.setattr(D, "_stream", lambda: None)
    with pytest.raises(ValueError, match="one GPU" if shapes[0] == (2, 5, 9, 9) and shapes[1:] == ((6, 5, 3, 3), (6,))
                       else "go together"):
        D.conv3x3(*(torch.zeros(s) for s in shapes))
