"""The kernels that a setting names are the ones that run: an explicit
wide-shard or run-time parameter family keeps every batch on its own kernels."""

import numpy as np
import pytest

import oracle
import synth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

from paper_2606_24417_amd.sbf import (VARIANT_AUTO, VARIANT_PARAM, VARIANT_ROLLING, VARIANT_WIDE,  # noqa: E402
                                      Filter)


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


def dev(x):
    return torch.from_numpy(np.array(x, copy=True)).cuda()


def doff(off):
    return dev(np.asarray(off, dtype=np.uint64).view(np.int64))


@pytest.mark.parametrize("S", [4, 16])
@pytest.mark.parametrize("variant,own", [(VARIANT_AUTO, False), (VARIANT_ROLLING, False), (VARIANT_WIDE, True),
                                         (VARIANT_PARAM, True)])
def test_explicit_families_do_not_bin(variant, own, S):
    """A binned insert of 50 Mbp keeps more than 200 MB of records."""
    d = dev(synth.background(50_000_000, 3))
    f = Filter(31, 28, 16, 4, 1 << 31, shard_words=S)
    f.variant = variant
    f.insert(d[:1000])
    torch.cuda.synchronize()
    before = torch.cuda.mem_get_info()[0]
    f.insert(d)
    torch.cuda.synchronize()
    kept = before - torch.cuda.mem_get_info()[0]
    f.close()
    assert (kept < 100 << 20) if own else (kept > 200 << 20)
