"""Loading pages: what a failed load leaves behind."""
import numpy as np
import pytest

from helpers import say
from paper_2607_16184_amd import pw, synth

pytestmark = pytest.mark.gpu

ENTRY = 24


def _entry_bits(L, index):
    return int(L.device_table()[index * ENTRY + 16])


def test_failed_load_leaves_the_entry_absent():
    """An error left pending by an earlier HIP call on the thread makes the load
    report PW_EHIP although its kernel ran: the slot goes back to the pool, so
    the device table must not name it. The block can then be loaded."""
    import torch
    from paper_2607_16184_amd.layer import PagedLayer
    cfg = synth.CONFIGS["tiny"]
    say("failed load")
    w16 = [synth.expert_weights(cfg, p) for p in range(3)]
    bits = [np.full((cfg.E, cfg.nrb(p)), 8, np.int32) for p in range(3)]
    L = PagedLayer(cfg, PagedLayer.pool_bytes_for(cfg, bits))
    rows = torch.from_numpy(w16[0][0].view(np.int16)).cuda()
    st = torch.cuda.current_stream().cuda_stream
    used = L.stats()
    torch.cuda.synchronize()
    assert pw._lib.hipSetDevice(1 << 20) != 0          # no such device: the call fails and is remembered
    with pytest.raises(pw.PWError) as ei:
        pw.pw_layer_load_page(L.handle, 0, 0, 0, 8, rows.data_ptr(), st)
    assert ei.value.status == pw.PW_EHIP
    torch.cuda.synchronize()
    assert not L.device_table()[:ENTRY].any()
    assert L.stats() == used
    pw.pw_layer_load_page(L.handle, 0, 0, 0, 8, rows.data_ptr(), st)
    torch.cuda.synchronize()
    assert _entry_bits(L, 0) == 8
    L.close()
