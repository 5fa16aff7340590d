"""Small networks store what the first modes of a larger one do and zeros in the padding,
byte for byte, in every storage form, and nothing past it: one to 32 samples per wave, waves that
are not full, odd numbers of samples."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

LD, GUARD = 128, 4096


def _modes(prec, E):
    """Mode of every byte of the stored amplitudes."""
    half = E + (E & 1) if prec.startswith("split1t") else E
    size = {"fp64": 8, "fp32": 4}.get(prec, 2)
    if prec in ("fp64", "fp32"):
        mode = np.tile(np.arange(LD), 2 * half)
    else:  # runs of 32 modes, two at a time (hi and lo values, or the columns of a pair)
        two = np.repeat(np.arange(LD).reshape(-1, 1, 32), 2, axis=1).reshape(-1)
        mode = np.tile(two, half if prec.startswith("split1t") else 2 * half)
    mode = np.repeat(mode, size)
    if prec == "split1t_f8":  # then the one-byte copies, in runs of 64
        two = np.repeat(np.arange(LD).reshape(-1, 1, 64), 2, axis=1).reshape(-1)
        mode = np.concatenate([mode, np.tile(two, half)])
    return mode


@pytest.mark.parametrize("prec", ["fp64", "fp32", "split_bf16", "split_fp16", "split1t_fp16", "split1t_f8"])
@pytest.mark.parametrize("M", [1, 3, 4, 5, 8, 15, 17, 33, 64])
@pytest.mark.parametrize("E", [1, 31, 65, 258])
def test_bytes_of_a_small_network(prec, M, E):
    import torch

    import paper_2503_12749_amd as mp
    r = torch.linspace(0.3, 1.2, 65, dtype=torch.float64, device="cuda")
    got = []
    for m in (M, 65):
        size = mp.mp_ab_bytes(m, E, prec)
        ab = torch.full((size + GUARD,), 0xA5, dtype=torch.uint8, device="cuda")
        n = torch.empty(E, dtype=torch.float64, device="cuda")
        mp.mp_sample(m, 9, E, r, 5, 0, prec, ab, n)
        ab = ab.cpu().numpy()
        assert np.all(ab[size:] == 0xA5)
        got.append(ab[:size])
    mode = _modes(prec, E)
    assert mode.size == got[0].size == got[1].size
    assert np.array_equal(got[0], np.where(mode < M, got[1], 0))
