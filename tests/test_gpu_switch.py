"""moe_set_channel_switch on its own: the row orders, their class counts and the
row-to-slot tables, entry by entry, against the definition (rows in stable order
of their source class)."""
import numpy as np
import pytest
import torch

from gpu_util import dev

pytestmark = pytest.mark.gpu

E = 3


class _Layer:
    """A descriptor with every row of every kind cached, and the tables that the
    switch writes."""

    def __init__(self, d, f):
        from paper_2503_21135_amd._lib import LayerDesc
        self.rows = (f, f, d)
        self.hdr = [np.stack([np.repeat(np.arange(E), R), np.tile(np.arange(R), E)], 1).astype(np.int32)
                    for R in self.rows]
        self.dhdr = [torch.from_numpy(h).to(dev()) for h in self.hdr]

        def table(n):
            return torch.full((n,), -7, dtype=torch.int32, device=dev())
        self.slot = [table(E * R) for R in self.rows]
        self.order_gu, self.order_dn, self.cnt = table(E * f), table(E * d), table(8 * E)
        self.staging = table(E * max(self.rows) + 1)
        D = self.desc = LayerDesc()
        D.n_experts, D.d_model, D.d_ff, D.group = E, d, f, 64
        for kind in range(3):
            D.kind[kind].n_slots = E * self.rows[kind]
            D.kind[kind].copy_hdr = self.dhdr[kind].data_ptr()
            D.kind[kind].copy_hdr_host = self.hdr[kind].ctypes.data
            D.kind[kind].row_slot = self.slot[kind].data_ptr()
        D.order_gu, D.order_dn = self.order_gu.data_ptr(), self.order_dn.data_ptr()
        D.class_cnt, D.staging = self.cnt.data_ptr(), self.staging.data_ptr()

    def check(self, on):
        on = [o.reshape(E, R) for o, R in zip(on, self.rows)]
        for kind, R in enumerate(self.rows):
            want = np.where(on[kind], np.arange(E * R).reshape(E, R), -1)
            assert np.array_equal(self.slot[kind].cpu().numpy().reshape(E, R), want)
        cnt = self.cnt.cpu().numpy().reshape(2, E, 4)
        for i, (cls, order) in enumerate(((on[0] + 2 * on[1], self.order_gu), (on[2] + 0, self.order_dn))):
            assert np.array_equal(order.cpu().numpy().reshape(E, -1), np.argsort(cls, 1, kind="stable"))
            assert np.array_equal(cnt[i], np.stack([(cls == c).sum(1) for c in range(4)], 1))


# rows below, at and past a wave (64), the workgroup's 16 waves (1024) and a
# wave's run of four 64-row steps (4096 rows in all)
@pytest.mark.parametrize("d,f", [(1, 63), (64, 65), (1023, 1024), (1025, 1408), (4096, 4097), (2048, 14336)])
def test_row_orders(d, f):
    import paper_2503_21135_amd as P
    L = _Layer(d, f)
    P.api.moe_set_channel_switch(L.desc, -1, None)
    on = [np.zeros(E * R, bool) for R in L.rows]
    L.check(on)
    rng = np.random.default_rng([d, f])
    for share in (0.05, 1.0, 0.5, 0.0):       # each on top of the one before
        for kind in (0, 2, 1):
            on[kind] = rng.random(E * L.rows[kind]) < share
            slots = rng.permutation(np.nonzero(on[kind])[0]).astype(np.int32)
            P.api.moe_set_channel_switch(L.desc, kind, slots)
            L.check(on)
