"""bsim_result_copy into memory that the caller names: device arrays at any
offset, pinned host memory given as device memory, and pageable host memory
given as device memory, which the runtime copies or refuses.  Results below and
above one MiB."""

import ctypes

import numpy as np
import pytest
import torch

from oracle import oracle as orc
from paper_2111_12493_amd import binding
from paper_2111_12493_amd import graphgen as gg

from gpu_util import assert_same, ctx

pytestmark = pytest.mark.gpu
FIELDS = binding.Result.FIELDS


def graph(n, m):
    rng = np.random.default_rng(n)
    return gg.from_edges(n, rng.integers(0, n, m), rng.integers(0, n, m), rng.integers(0, 5, m),
                         types=[[int(t)] for t in rng.integers(0, 4, n)])


def copied(r, field, address, kind):
    return binding.lib().bsim_result_copy(r.ptr, field.encode(), ctypes.c_void_p(address), kind)


@pytest.fixture(scope="module", params=[(1, 1), (900, 4001), (150001, 400003)])
def result(request):
    g = graph(*request.param)
    r = binding.summarize(ctx(), binding.DeviceGraph(g), k_max=2, stop_at_fixpoint=False)
    ref = r.to_dict()
    assert_same(ref, orc.summarize(g, 2, False), request.param)
    yield r, ref
    r.free()


@pytest.mark.parametrize("field", sorted(FIELDS))
@pytest.mark.parametrize("shift", [0, 1, 4, 12])
def test_device_arrays_at_any_offset(result, field, shift):
    r, ref = result
    want = ref[field].view(np.uint8)
    a = torch.full((want.size + 64,), 0xA5, dtype=torch.uint8, device="cuda")
    assert copied(r, field, a.data_ptr() + 16 + shift, binding.MEM_DEVICE) == binding.OK
    got = a.cpu().numpy()
    assert np.array_equal(got[16 + shift:16 + shift + want.size], want)
    assert (got[:16 + shift] == 0xA5).all() and (got[16 + shift + want.size:] == 0xA5).all()


@pytest.mark.parametrize("field", sorted(FIELDS))
def test_pinned_memory_given_as_device_memory(result, field):
    r, ref = result
    want = ref[field].view(np.uint8)
    a = torch.zeros(want.size + 8, dtype=torch.uint8, pin_memory=True)
    assert copied(r, field, a.data_ptr(), binding.MEM_DEVICE) == binding.OK
    assert np.array_equal(a.numpy()[:want.size], want)


@pytest.mark.parametrize("field", sorted(FIELDS))
def test_pageable_memory_given_as_device_memory(result, field):
    r, ref = result
    want = ref[field]
    a = np.zeros(want.size + 8, dtype=want.dtype)
    rc = copied(r, field, a.ctypes.data, binding.MEM_DEVICE)
    assert rc in (binding.OK, binding.E_DEVICE)
    if rc == binding.OK:
        assert np.array_equal(a[:want.size], want)
    # and the result is still whole
    assert np.array_equal(r.fetch(field), want)
