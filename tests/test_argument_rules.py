"""The one-shot attention call has its argument rules twice: once in a single pass that only says yes or no, once with the
words of a refusal.  They may not drift apart: whatever the first takes the second takes too, and gives the same arguments, for every
way in which an argument can be off.  (Stand-ins for tensors: the rules look at properties only.)"""
import itertools

import numpy as np
import pytest
import torch

from paper_2509_25401_amd import binding

B, H, L, D, BQ, BK = 2, 3, 700, 64, 64, 128
SHAPES = {"Q": (B, H, L, D), "K": (B, H, L, D), "V": (B, H, L, D), "cache_flags": (B, H, 11), "kv_mask": (B, H, 11, 1),
          "O_cache": (B, H, L, D), "O": (B, H, L, D)}
SYMBOLS = ("cache_flags", "kv_mask")
OPTIONAL = SYMBOLS + ("O_cache",)


class Tensor:
    def __init__(self, name):
        self.shape, self.dtype = torch.Size(SHAPES[name]), torch.uint8 if name in SYMBOLS else torch.bfloat16
        self.device, self.contiguous, self.address = torch.device("cuda", 0), True, 4096 * (1 + list(SHAPES).index(name))

    is_cuda = property(lambda self: self.device.type == "cuda")
    dim = lambda self: len(self.shape)
    get_device = lambda self: self.device.index if self.is_cuda else -1
    is_contiguous = lambda self: self.contiguous
    data_ptr = lambda self: self.address


def resized(axis, by):
    def change(t):
        if axis < len(t.shape):
            t.shape = torch.Size(n + by * (i == axis) for i, n in enumerate(t.shape))
    return change


CHANGES = {
    "float32": lambda t: setattr(t, "dtype", torch.float32),
    "bool": lambda t: setattr(t, "dtype", torch.bool),
    "uint8": lambda t: setattr(t, "dtype", torch.uint8),
    "strided": lambda t: setattr(t, "contiguous", False),
    "other GPU": lambda t: setattr(t, "device", torch.device("cuda", 1)),
    "host": lambda t: setattr(t, "device", torch.device("cpu")),
    "flat": lambda t: setattr(t, "shape", torch.Size([t.shape.numel()])),
    "one more axis": lambda t: setattr(t, "shape", torch.Size(t.shape) + (1,)),
    **{f"axis {a} by {by}": resized(a, by) for a in range(4) for by in (-1, 1)},
}


def both(args):
    """(single pass, or None) and (checks, or None where they refuse)"""
    given = all(args[n] is not None for n in ("Q", "K", "V", "O"))     # the caller sends the others to the checks
    quick = binding._fwd_args_valid(**args) if given else None
    try:
        checked = binding._fwd_args(**args)
    except ValueError:
        checked = None
    return quick, checked


def arguments(**blocks):
    return dict({n: Tensor(n) for n in SHAPES}, **{"block_q": BQ, "block_k": BK, **blocks})


@pytest.mark.parametrize("change", sorted(CHANGES))
def test_single_pass_and_checks_agree_on_every_change(change):
    for names in itertools.chain.from_iterable(itertools.combinations(SHAPES, n) for n in (1, 2, 7)):
        args = arguments()
        for n in names:
            CHANGES[change](args[n])
        quick, checked = both(args)
        assert (quick is None) == (checked is None), names
        assert quick is None or list(quick) == checked


@pytest.mark.parametrize("left_out", [c for n in range(4) for c in itertools.combinations(OPTIONAL, n)] + [("O",)])
def test_arguments_left_out(left_out):
    quick, checked = both(dict(arguments(), **{n: None for n in left_out}))
    assert (quick is None) == (checked is None) == (not set(left_out) <= set(OPTIONAL))
    assert quick is None or list(quick) == checked


@pytest.mark.parametrize("block_q,block_k", [(64, 64), (63, 128), (64, 88), (128, 128), (0, 128), (-64, 128), (64, 0), (np.int64(64), 128),
                                             (64, np.int32(128)), (64.0, 128), (True, 128)])
def test_block_sizes(block_q, block_k):
    """Whole numbers of other types go through the checks and come out the same."""
    quick, checked = both(arguments(block_q=block_q, block_k=block_k))
    if type(block_q) is int and type(block_k) is int:
        assert (quick is None) == (checked is None)
    assert quick is None or list(quick) == checked


def test_output_as_cache():
    args = arguments()
    args["O_cache"] = args["O"]
    quick, checked = both(args)
    assert list(quick) == checked
