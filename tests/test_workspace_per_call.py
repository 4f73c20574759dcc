"""A layer's workspace belongs to one call: nothing of it is kept between calls, so that graphs captured at several
batch sizes, streams and threads may share a layer."""
import numpy as np
import pytest
import torch

from paper_1805_12549_amd import binding as B
from paper_1805_12549_amd import workloads as W


class _FakeLib:
    """cg_conv_forward that notes its workspace; while it runs, a second call of the same layer is made."""

    def __init__(self):
        self.layer, self.seen, self.live = None, [], set()

    def cg_conv_forward(self, handle, n, x, residual, y, bitmap, counts, workspace, workspace_bytes, stream):
        assert workspace % 256 == 0 and workspace_bytes >= 1000 * n
        self.seen.append(workspace)
        if len(self.seen) == 1:
            self.layer.forward(torch.zeros(n, 4), y=torch.zeros(1), bitmap=False, counts=False)
        return B.CG_OK

    def alloc(self, size, stream):
        assert size > 0 and stream == 77
        p = 4096 * (1 + len(self.seen))
        assert p not in self.live
        self.live.add(p)
        return p

    def free(self, p):
        self.live.remove(p)


def test_two_calls_at_once_have_workspaces_of_their_own(monkeypatch):
    fake = _FakeLib()
    monkeypatch.setattr(B, "_lib", fake)
    monkeypatch.setattr(B, "_raw_alloc", fake.alloc, raising=False)
    monkeypatch.setattr(B, "_raw_free", fake.free, raising=False)
    monkeypatch.setattr(B, "cg_conv_workspace_bytes", lambda handle, n: 1000 * n)
    monkeypatch.setattr(B.GatedConv, "_stream_ptr", lambda self: 77)
    layer = object.__new__(B.GatedConv)
    layer.__dict__.update(_torch=torch, handle=0, _ws=None, _ws_need={}, ho=2, wo=2, c_out=8, words=1)
    fake.layer = layer
    layer.forward(torch.zeros(3, 4), y=torch.zeros(1), bitmap=False, counts=False)
    assert len(fake.seen) == 2 and fake.seen[0] != fake.seen[1]
    assert not fake.live                                              # given back


def _layer(n_max):
    """256 channels at 14x14: one or two images split K over workgroups, whose sums go through the workspace."""
    shape = W.LayerShape("ws_256@14", n_max, 14, 14, 256, 256)
    q = W.quantize_int8(W.make_inputs(shape, 9700, kind="coherent", rho=0.35))
    thr = W.calibrate_gate_int8(q, 0.35, sample_images=None)
    dev = lambda a: torch.from_numpy(a).cuda()
    layer = B.GatedConv(n_max=n_max, h=14, w=14, c_in=256, c_out=256, c_base=shape.c_base, w_base=dev(q.w_base),
                        w_cond=dev(q.w_cond), in_dtype=B.CG_I8, out_dtype=B.CG_I32, gate_thr_i32=thr)
    return layer, dev(q.x)


@pytest.mark.gpu
def test_a_graph_of_one_batch_size_survives_calls_of_another():
    layer, x = _layer(8)
    want = {n: layer.forward(x[:n])[0].clone() for n in (1, 2, 3)}
    side = torch.cuda.Stream()
    graphs = {}
    for n in (1, 2):
        side.wait_stream(torch.cuda.current_stream())
        with torch.cuda.stream(side):
            layer.forward(x[:n])
            torch.cuda.synchronize()
            g = torch.cuda.CUDAGraph()
            with torch.cuda.graph(g, stream=side):
                graphs[n] = (g, layer.forward(x[:n])[0])
        torch.cuda.synchronize()
        # a larger batch, then tensors of every size a workspace could have had: what was given back is in use again
        assert torch.equal(layer.forward(x[:3])[0], want[3])
        others = [torch.full((size,), 91, dtype=torch.uint8, device="cuda") for size in (1 << 20, 2 << 20, 4 << 20, 8 << 20) for _ in range(4)]
        for m, (gm, ym) in graphs.items():
            for _ in range(3):
                ym.zero_()
                gm.replay()
                assert torch.equal(ym, want[m])
                assert torch.equal(layer.forward(x[:3])[0], want[3])
        assert all(int((t != 91).sum()) == 0 for t in others)
    layer.close()


@pytest.mark.gpu
def test_one_layer_on_two_streams():
    layer, x = _layer(4)
    want = [layer.forward(x[i:i + 1])[0].clone() for i in range(4)]
    torch.cuda.synchronize()
    streams = [torch.cuda.Stream() for _ in range(2)]
    got = []
    for k in range(40):
        for i, s in enumerate(streams):
            with torch.cuda.stream(s):
                got.append(((2 * k + i) % 4, layer.forward(x[(2 * k + i) % 4:(2 * k + i) % 4 + 1])[0]))
    torch.cuda.synchronize()
    assert all(torch.equal(y, want[i]) for i, y in got)
    layer.close()
