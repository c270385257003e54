"""Both forward passes of a call, side by side or one after the other: one result, whatever the size and the stream."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


# small calls, with one stream, and many tokens through one layer and two
@pytest.mark.parametrize("layers,hidden,batch,seq", [(1, 64, 1, 8), (3, 128, 1, 8), (1, 320, 2, 23), (1, 384, 2, 23), (1, 256, 32, 128), (2, 128, 8, 128)])
def test_both_passes_equal_single_passes(layers, hidden, batch, seq):
    import torch
    from paper_2109_15082_amd import binding as B
    rng = np.random.default_rng(hidden)
    mod = B.MremModule(layers, hidden, hidden // 64, 4 * hidden, batch, seq)
    mod.teacher.copy_(torch.from_numpy(rng.standard_normal(mod.teacher.numel(), dtype=np.float32) * np.float32(0.02)))
    B.mrem_teacher_prepare(mod.ctx, mod.teacher, mod.teacher_cache)
    mod.params.copy_(mod.teacher)
    mod.init_steps()
    x = torch.from_numpy(rng.standard_normal((batch, seq, hidden), dtype=np.float32)).cuda().bfloat16()
    mod.calibrate(x)
    f_fp, f_q = (f.clone() for f in mod.forward(x, x))
    B.mrem_profile_gemm_begin(mod.ctx)  # times each product, on one stream
    g_fp, g_q = (g.clone() for g in mod.forward(x, x))
    B.mrem_profile_gemm_end(mod.ctx)
    assert torch.equal(f_fp, g_fp) and torch.equal(f_q, g_q)
    # while the caller's stream is captured: replays repeat the eager results
    out_fp, out_q = mod.new_outputs(batch, seq)
    side = torch.cuda.Stream()
    graph = torch.cuda.CUDAGraph()
    torch.cuda.synchronize()
    with torch.cuda.graph(graph, stream=side):
        mod.forward(x, x, None, out_fp, out_q)
    for _ in range(3):
        out_fp.zero_()
        out_q.zero_()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(out_fp, f_fp) and torch.equal(out_q, f_q)
        h_fp, h_q = mod.forward(x, x)
        assert torch.equal(h_fp, f_fp) and torch.equal(h_q, f_q)


def _forked_module(torch, B):
    rng = np.random.default_rng(3)
    mod = B.MremModule(3, 768, 12, 3072, 16, 64)
    mod.teacher.copy_(torch.from_numpy(rng.standard_normal(mod.teacher.numel(), dtype=np.float32) * np.float32(0.02)))
    B.mrem_teacher_prepare(mod.ctx, mod.teacher, mod.teacher_cache)
    mod.params.copy_(mod.teacher)
    mod.init_steps()
    x = torch.from_numpy(rng.standard_normal((16, 64, 768), dtype=np.float32)).cuda().bfloat16()
    mod.calibrate(x)
    return mod, x


def test_outputs_in_place_of_an_input():
    """The quantized pass's outputs start at the input that both passes read; and its input lies in the other's outputs."""
    import torch
    from paper_2109_15082_amd import binding as B
    mod, x = _forked_module(torch, B)
    f_fp, f_q = (f.clone() for f in mod.forward(x, x))
    out_fp, out_q = mod.new_outputs(16, 64)
    for _ in range(3):
        out_q[0].copy_(x)
        mod.forward(out_q[0], out_q[0], None, out_fp, out_q)
        assert torch.equal(out_fp, f_fp) and torch.equal(out_q, f_q)
    g_fp, g_q = (f.clone() for f in mod.forward(x, f_fp[1].clone()))
    for _ in range(3):
        out_fp.zero_()
        mod.forward(x, out_fp[1], None, out_fp, out_q)
        assert torch.equal(out_fp, g_fp) and torch.equal(out_q, g_q)


@pytest.mark.parametrize("own_streams", [True, False])
def test_two_callers_on_one_context(own_streams):
    """Two threads with a workspace and outputs each, on two streams and on one, repeat what one caller gets."""
    import threading
    import torch
    from paper_2109_15082_amd import binding as B
    mod, x = _forked_module(torch, B)
    xs = [x, (x.float() * 0.5 + 0.1).bfloat16()]
    ref = [tuple(f.clone() for f in mod.forward(v, v)) for v in xs]
    streams = [torch.cuda.Stream() for _ in xs] if own_streams else [torch.cuda.Stream()] * 2
    spaces = [torch.empty_like(mod.workspace) for _ in xs]
    torch.cuda.synchronize()
    got = [[] for _ in xs]

    def call(i):
        with torch.cuda.stream(streams[i]):
            for _ in range(8):
                fp, q = mod.new_outputs(16, 64)
                B.mrem_module_forward(mod.ctx, mod.params, mod.teacher, mod.teacher_cache, xs[i], xs[i], None, 16, 64, fp, q, spaces[i])
                got[i].append((fp, q))
    threads = [threading.Thread(target=call, args=(i,)) for i in range(2)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    torch.cuda.synchronize()
    for i in range(2):
        assert len(got[i]) == 8
        for fp, q in got[i]:
            assert torch.equal(fp, ref[i][0]) and torch.equal(q, ref[i][1])


def test_more_callers_streams_than_are_served():
    """Calls from more streams than the library keeps streams for take over those that are idle."""
    import torch
    from paper_2109_15082_amd import binding as B
    mod, x = _forked_module(torch, B)
    f_fp, f_q = (f.clone() for f in mod.forward(x, x))
    torch.cuda.synchronize()
    for _ in range(20):
        with torch.cuda.stream(torch.cuda.Stream()):
            g_fp, g_q = mod.forward(x, x)
        torch.cuda.synchronize()
        assert torch.equal(g_fp, f_fp) and torch.equal(g_q, f_q)


def test_streams_stay_sound_when_busy_and_when_given_back():
    """More callers' streams than the library keeps, all with work queued; then contexts that end, the last one among them."""
    import gc
    import torch
    from paper_2109_15082_amd import binding as B
    gc.collect()
    for _ in range(3):
        mod, x = _forked_module(torch, B)
        f_fp, f_q = (f.clone() for f in mod.forward(x, x))
        streams = [torch.cuda.Stream() for _ in range(20)]
        spaces = [torch.empty_like(mod.workspace) for _ in streams]
        outs = [mod.new_outputs(16, 64) for _ in streams]
        torch.cuda.synchronize()
        for _ in range(2):
            for st, ws, (fp, q) in zip(streams, spaces, outs):
                with torch.cuda.stream(st):
                    B.mrem_module_forward(mod.ctx, mod.params, mod.teacher, mod.teacher_cache, x, x, None, 16, 64, fp, q, ws)
        mod.close()  # work may still be queued
        torch.cuda.synchronize()
        for fp, q in outs:
            assert torch.equal(fp, f_fp) and torch.equal(q, f_q)


# on both sides of the lines from which on the full-precision pass gets a stream of its own
@pytest.mark.parametrize("layers,hidden,batch,seq", [(10, 64, 1, 8), (9, 64, 1, 8), (2, 256, 1, 64), (2, 256, 1, 63), (3, 128, 3, 128), (3, 128, 1, 383),
                                                     (1, 512, 16, 128), (4, 64, 8, 128), (2, 128, 32, 128)])
def test_both_passes_equal_single_passes_around_the_rule(layers, hidden, batch, seq):
    test_both_passes_equal_single_passes(layers, hidden, batch, seq)
