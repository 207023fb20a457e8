"""Scratch memory of the kernels that every default step runs (host-only check
of the compiler's remarks for gfx950): none, but for the instantiations listed
here with the bytes per lane that they spill.  One that is not listed, or spills
more, has lost registers."""
import re

import pytest

from test_kernel_resources import _resource_usage

# source, kernels expected in it, {template arguments of a kernel: bytes per lane}
STEP = [
    ("fdm.hip", 40, {
        "k_fdm_xy_fwd<3,1>": 20,   # in-plane pass of axes of 65 to 96 nodes, capped at 168 registers so that
        "k_fdm_xy_fwd<3,0>": 12,   # two blocks of six waves share a compute unit
    }),
    ("products.hip", 20, {
        "k_nt<4,2,1>": 92,         # 97 to 128 orbitals: 16 accumulator tiles a wave
        "k_nt<4,2,0>": 32,
        "k_nn<3>": 28,             # 33 to 48 orbitals
        "k_nn<7>": 12,             # 97 to 112
        "k_nn<8>": 28,             # 113 to 128
    }),
    ("octant.hip", 40, {
        "k_oct_moments<7>": 124,   # multipole orders above the default 6: 14 and 17 accumulator tiles
        "k_oct_moments<8>": 340,
    }),
    ("lowdin.hip", 3, {}),
]


def _name(mangled):
    """k_name<template arguments> of a mangled kernel of namespace fsic."""
    m = re.match(r"_ZN4fsic\d+(k_\w+?)(?:I((?:L[ib]\d+E)+)E)?E", mangled)
    if not m:
        return mangled
    return m.group(1) + ("<" + ",".join(re.findall(r"L[ib](\d+)E", m.group(2))) + ">" if m.group(2) else "")


@pytest.mark.parametrize("source,kernels,known", STEP, ids=[s[0] for s in STEP])
def test_scratch_is_as_listed(source, kernels, known):
    usage = {_name(k): v.get("ScratchSize") for k, v in _resource_usage(source).items()}
    assert len(usage) >= kernels and set(known) <= set(usage), sorted(usage)
    over = {k: v for k, v in usage.items() if v is None or v > known.get(k, 0)}
    assert not over, over
