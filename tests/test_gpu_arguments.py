"""The one-shot attention call takes its arguments for valid first and checks them one by one only if they are not: what
the checks refuse is refused with the same words."""
import pytest
import torch

import paper_2509_25401_amd as pkg
from paper_2509_25401_amd import binding

pytestmark = pytest.mark.gpu

B, H, L, D, BQ, BK = 1, 2, 256, 64, 64, 128


def arguments():
    t = {name: torch.zeros(B, H, L, D, dtype=torch.bfloat16, device="cuda") for name in ("Q", "K", "V", "O", "O_cache")}
    t["cache_flags"] = torch.zeros(B, H, L // BQ, dtype=torch.uint8, device="cuda")
    t["kv_mask"] = torch.zeros(B, H, L // BQ, 1, dtype=torch.uint8, device="cuda")
    return dict(t, block_q=BQ, block_k=BK)


WRONG = {
    "dtype": lambda a, n: a[n].to(torch.int32) if n in ("cache_flags", "kv_mask") else a[n].float(),
    "shape": lambda a, n: torch.cat([a[n], a[n]], dim=1),
    "stride": lambda a, n: a[n].transpose(1, 2).contiguous().transpose(1, 2),
    "device": lambda a, n: a[n].cpu(),
}


@pytest.mark.parametrize("name", ["Q", "K", "V", "O", "O_cache", "cache_flags", "kv_mask"])
@pytest.mark.parametrize("how", sorted(WRONG))
def test_wrong_argument_is_refused_with_the_words_of_the_checks(name, how):
    print(f"[case] argument {name} wrong in {how}", flush=True)
    args = arguments()
    args[name] = WRONG[how](args, name)
    with pytest.raises(ValueError) as want:
        binding._fwd_args(**args)
    with pytest.raises(ValueError) as got:
        pkg.sparse_attn_fwd(**args)
    assert str(got.value) == str(want.value)


@pytest.mark.parametrize("change", [{"O_cache": None}, {"cache_flags": None, "O_cache": None}, {"kv_mask": None}, {"O_cache": "O"}])
def test_both_ways_give_the_same_arguments(change):
    args = arguments()
    for name, value in change.items():
        args[name] = args["O"] if value == "O" else value
    pkg.sparse_attn_fwd(**args)
    assert list(binding._fwd_args_valid(**args)) == binding._fwd_args(**args)
