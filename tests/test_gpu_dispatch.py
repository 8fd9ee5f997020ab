"""GPU parity of the Dispatch step (include/mux_dispatch.h) against its oracle: bit-exact placement of the tasks' packed
tokens on the rows of the aligned batch and back, bf16 and fp32 elements, vector and element-wise paths."""
import numpy as np
import pytest

from oracle import dispatch as odisp
from oracle import segtab

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def env():
    import torch
    import paper_2603_02885_amd as mx
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    mx.load_library()
    return mx, torch


@pytest.mark.parametrize("flags", [0, 1])
@pytest.mark.parametrize("width,elem", [(64, 2), (40, 4), (13, 2), (257, 4), (4096, 2)])
def test_gather_scatter_bit_exact(env, width, elem, flags):
    mx, torch = env
    rng = np.random.default_rng(width + 7 * elem + flags)
    n_tasks = 37                                                       # more than one batch of task pointers
    lens = [[int(v) for v in rng.integers(1, 90, size=int(rng.integers(0, 4)))] for _ in range(n_tasks)]
    lens[3] = [200, 1, 64]
    chunk = 32
    ot = segtab.build(lens, chunk, 128, flags)
    st = mx.mux_segtab_build([mx.TaskDesc(mx.MUX_ADAPTER_NONE, 0, 1.0, l) for l in lens], chunk, 128, flags)
    assert np.array_equal(mx.mux_segtab_serialize(st), ot.image)
    dev = "cuda:0"
    nb = mx.mux_segtab_device_bytes(st)
    dtab = torch.zeros(nb, dtype=torch.uint8, device=dev)
    mx.mux_segtab_upload(st, dtab, nb)
    tdt = torch.bfloat16 if elem == 2 else torch.float32
    print(f"dispatch case: T={ot.T} width={width} elem={elem} flags={flags}", flush=True)
    # small integers: exact in bf16 and fp32, so the comparison is bitwise
    srcs = [rng.integers(-120, 120, size=(sum(l), width)).astype(np.float64) for l in lens]
    ld_task, ld_al = width + (8 if width % 8 == 0 else 3), width + (16 if width % 8 == 0 else 1)
    tsrc = [torch.zeros((max(s.shape[0], 1), ld_task), dtype=tdt, device=dev) for s in srcs]
    for t, s in zip(tsrc, srcs):
        if s.shape[0]:
            t[:s.shape[0], :width] = torch.from_numpy(s).to(dev).to(tdt)
    aligned = torch.full((ot.T, ld_al), float("nan"), dtype=tdt, device=dev)
    ptrs = [t if s.shape[0] else None for t, s in zip(tsrc, srcs)]
    mx.mux_dispatch_gather(st, dtab, ptrs, ld_task, aligned, ld_al, width, elem, torch.cuda.current_stream())
    torch.cuda.synchronize()
    got = aligned[:, :width].float().cpu().numpy().astype(np.float64)
    want = odisp.gather(srcs, ot.row_task, width)
    assert np.array_equal(got, want)
    assert torch.isnan(aligned[:, width:]).all()                       # nothing written beyond the width
    # scatter back into fresh buffers
    tdst = [torch.full((max(s.shape[0], 1), ld_task), float("nan"), dtype=tdt, device=dev) for s in srcs]
    mx.mux_dispatch_scatter(st, dtab, aligned, ld_al, [t if s.shape[0] else None for t, s in zip(tdst, srcs)], ld_task,
                            width, elem, torch.cuda.current_stream())
    torch.cuda.synchronize()
    back = odisp.scatter(want, ot.row_task, n_tasks)
    for t, s, b in zip(tdst, srcs, back):
        if s.shape[0]:
            assert np.array_equal(t[:s.shape[0], :width].float().cpu().numpy().astype(np.float64), b)
            assert torch.isnan(t[:s.shape[0], width:]).all()


def test_rows_past_the_caches(env):
    """More bytes than are read through the caches (112 MB), odd sequence lengths and padding rows: a gather and a scatter,
    bit by bit against the rows that the table gives."""
    mx, torch = env
    width, chunk, dev = 3080, 64, "cuda:0"
    lens = [[4099, 77, 1], [6001, 333], [2050] * 3, [3001]]
    st = mx.mux_segtab_build([mx.TaskDesc(mx.MUX_ADAPTER_NONE, 0, 1.0, l) for l in lens], chunk, 0, 0)
    T = mx.mux_segtab_rows(st)
    assert T * width * 2 > 112 << 20
    nb = mx.mux_segtab_device_bytes(st)
    dtab = torch.zeros(nb, dtype=torch.uint8, device=dev)
    mx.mux_segtab_upload(st, dtab, nb)
    gen = torch.Generator(device=dev).manual_seed(5)
    src = [torch.randint(-2 ** 15, 2 ** 15 - 1, (sum(l), width), device=dev, generator=gen, dtype=torch.int32).to(torch.int16) for l in lens]
    aligned = torch.full((T, width), -1, dtype=torch.int16, device=dev)
    print(f"dispatch case: T={T} width={width}", flush=True)
    mx.mux_dispatch_gather(st, dtab, src, width, aligned, width, width, 2, torch.cuda.current_stream())
    row_task = torch.from_numpy(np.ascontiguousarray(mx.mux_segtab_row_task(st))).to(dev)
    torch.cuda.synchronize()
    for t, s in enumerate(src):
        assert torch.equal(aligned[row_task == t], s), t
    assert not aligned[row_task < 0].any()
    back = [torch.full_like(s, -1) for s in src]
    mx.mux_dispatch_scatter(st, dtab, aligned, width, back, width, width, 2, torch.cuda.current_stream())
    torch.cuda.synchronize()
    for t, s in enumerate(src):
        assert torch.equal(back[t], s), t


def test_argument_checks(env):
    mx, torch = env
    st = mx.mux_segtab_build([mx.TaskDesc(mx.MUX_ADAPTER_NONE, 0, 1.0, [5])], 16, 0, 0)
    nb = mx.mux_segtab_device_bytes(st)
    dtab = torch.zeros(nb, dtype=torch.uint8, device="cuda:0")
    mx.mux_segtab_upload(st, dtab, nb)
    x = torch.zeros((16, 8), dtype=torch.bfloat16, device="cuda:0")
    with pytest.raises(mx.MuxError):
        mx.mux_dispatch_gather(st, dtab, [x], 8, x, 8, 8, 3)            # element size
    with pytest.raises(mx.MuxError):
        mx.mux_dispatch_gather(st, dtab, [x], 4, x, 8, 8, 2)            # leading dimension below the width
    with pytest.raises(mx.MuxError):
        mx.mux_dispatch_gather(st, dtab, [None], 8, x, 8, 8, 2)         # a task with tokens and no buffer
