"""GPU parity: forward and backward vs the float64 oracle, element by element, through the C ABI."""
import time

import numpy as np
import pytest
import torch

from oracle import mate_oracle as orc
from paper_2109_04312_amd import synth
from tests import helpers as hp

pytestmark = pytest.mark.gpu
ROW, COL = synth.HEAD_ROW, synth.HEAD_COL


def small_workload(seed, dtype, B=2, N=200, H=4, bwd=True, **kw):
    rng = np.random.default_rng(seed)
    st = synth.random_structure(rng, B, N, **kw)
    q, k, v, do = synth.draw_tensors(rng, B, H, N, 64, dtype, 4)
    hk = np.array([ROW, COL] * (H // 2), np.uint8)
    return synth.Workload(f"small{seed}", dtype, st, hk, q, k, v, do if bwd else None, 0.125)


def check_workload(w, backward, pairs=None, label=""):
    print(f"case {label or w.name} dtype={w.dtype} shape={w.shape} bwd={backward}", flush=True)
    got, seg = hp.run_hip(w, backward)
    hp.compare_segments(seg, w.structure)
    t0 = time.perf_counter()
    ref = hp.run_oracle(w, backward, pairs)
    print(f"   oracle: {len(ref)} (sequence, head) pairs in {time.perf_counter() - t0:.1f} s", flush=True)
    worst = hp.compare(got, ref, w, label or w.name)
    print(hp.report(worst), flush=True)


def test_config1_tiny_f32_forward():
    check_workload(synth.make_config(1), backward=False)


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("seed", [0, 1, 2])
def test_small_scattered_fwd_bwd(seed, dtype):
    w = small_workload(seed, dtype, N=[200, 333, 130][seed], max_rows=12, max_cols=7, max_global=20,
                       max_cell=4, scatter=seed != 0, sparse_ids=seed == 2)
    check_workload(w, backward=True)


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_degenerate_structures(dtype):
    """All pad, all global (dense), no globals, one row, one column, single tokens."""
    L, G, P = synth.TOK_LOCAL, synth.TOK_GLOBAL, synth.TOK_PAD
    N = 150
    rng = np.random.default_rng(12)
    flags = np.full((7, N), L, np.uint8)
    row = rng.integers(0, 9, (7, N)).astype(np.int32)
    col = rng.integers(0, 4, (7, N)).astype(np.int32)
    flags[0] = P                                   # empty sequence
    flags[1] = G                                   # dense attention
    flags[1, 100:] = P
    row[3] = 5                                     # one row, no globals  (flags[2]: generic, no globals)
    col[4] = 1                                     # one column
    flags[4, :3] = G
    flags[5] = P                                   # a single table token
    flags[5, 77] = L
    flags[6] = P                                   # one global + one local
    flags[6, 3] = G
    flags[6, 140] = L
    st = synth.Structure(row, col, flags)
    q, k, v, do = synth.draw_tensors(rng, 7, 2, N, 64, dtype, 4)
    w = synth.Workload("degenerate", dtype, st, np.array([ROW, COL], np.uint8), q, k, v, do, 0.125)
    check_workload(w, backward=True)


@pytest.mark.parametrize("n_global,N", [(200, 2048), (700, 1500), (1024, 1024), (129, 4000)])
def test_many_question_tokens(n_global, N):
    """Question-token owners spanning several 128-row tiles, with and without chunked streams
    (the all-question case is plain dense attention)."""
    rng = np.random.default_rng(n_global)
    R, C = 60, 5
    row, col, flag = synth.flatten_table(N, n_global, R, C, synth.geometric_lengths(rng, 4.0, 12, R * C))
    st = synth.Structure(row[None], col[None], flag[None])
    q, k, v, do = synth.draw_tensors(rng, 1, 2, N, 64, "bf16", 4)
    w = synth.Workload(f"globals{n_global}", "bf16", st, np.array([ROW, COL], np.uint8), q, k, v, do, 0.125)
    check_workload(w, backward=True)


def test_maximum_sequence_length():
    """N = 16384, the largest length the library accepts (the segment builder's LDS limit): a
    full 128-tile owner grid, 9-bit and 10-bit ids, a sequence filled to the last position."""
    N = 16384
    rng = np.random.default_rng(16384)
    R, C = 700, 12
    row, col, flag = synth.flatten_table(N, 100, R, C, synth.geometric_lengths(rng, 2.0, 8, R * C))
    assert (flag != synth.TOK_PAD).all()      # the table is cut at N: no padding at all
    st = synth.Structure(row[None], col[None], flag[None])
    q, k, v, do = synth.draw_tensors(rng, 1, 2, N, 64, "bf16", 4)
    w = synth.Workload("max_length", "bf16", st, np.array([ROW, COL], np.uint8), q, k, v, do, 0.125)
    check_workload(w, backward=True)


def test_config2_bf16_fwd_bwd():
    check_workload(synth.make_config(2), backward=True)


def test_config3_bf16_fwd_bwd():
    # 64 of the 128 (sequence, head) pairs: every sequence, four row heads and four column heads
    w = synth.make_config(3)
    pairs = [(b, h) for b in range(8) for h in (0, 1, 6, 7, 8, 9, 14, 15)]
    check_workload(w, backward=True, pairs=pairs)


@pytest.mark.parametrize("b,kind", [(0, ROW), (0, COL), (1, ROW), (1, COL)])
def test_config4_headline_every_head(b, kind):
    # Full benchmark size, the launch configuration bench.py times: every one of the 32
    # (sequence, head) pairs is compared with the oracle element by element, eight per test (one
    # sequence's row heads or column heads; the oracle takes 1.5 - 6 s per pair at this length).
    w = synth.make_config(4)
    pairs = [(b, h) for h in range(16) if w.head_kind[h] == kind]
    assert len(pairs) == 8
    check_workload(w, backward=True, pairs=pairs, label=f"{w.name} b={b} kind={kind}")


def test_config5_ragged_sampled_heads():
    # every sequence with one row head and one column head (32 of the 256 pairs);
    # b=0: one-row table (row heads dense), b=1: one-column table (column heads dense)
    w = synth.make_config(5)
    pairs = [(b, h) for b in range(16) for h in (b % 8, 8 + (3 * b) % 8)]
    check_workload(w, backward=True, pairs=pairs)


def test_config6_long_cells_sampled_heads():
    # long expanded cells: both views have segments of hundreds of tokens; every sequence, two
    # row heads and two column heads (32 of the 128 pairs)
    w = synth.make_config(6)
    check_workload(w, backward=True, pairs=[(b, h) for b in range(8) for h in (0, 5, 8, 15)])


@pytest.mark.parametrize("idx", [4, 5])
def test_full_size_properties_over_all_heads(idx):
    """Invariants that need no oracle, checked on EVERY (sequence, head) of the full-size
    configurations (the oracle comparison above covers a sample of them):
      * V = 1 everywhere  =>  O = 1 at every non-pad position (each softmax row sums to 1);
      * sum_j dV_j = sum_k dO_k over non-pad tokens (same reason);
      * sum_j dK_j = 0 (every row of dS sums to 0)."""
    from paper_2109_04312_amd import mate
    w = synth.make_config(idx)
    r, c, f = hp.dev_structure(w.structure)
    seg = mate.build_segments(r, c, f)
    q, k, v, do = (hp.to_dev(x, "bf16") for x in (w.q, w.k, w.v, w.do))
    nonpad = (f != synth.TOK_PAD)[:, None, :, None]
    ones = torch.ones_like(v)
    o1, _ = mate.attn_fwd(q, k, ones, seg, w.head_kind, w.scale)
    assert float(((o1.float() - 1.0).abs() * nonpad).max()) <= 4e-3      # one bf16 ulp at 1
    out, lse = mate.attn_fwd(q, k, v, seg, w.head_kind, w.scale)
    dq, dk, dv = mate.attn_bwd(q, k, v, out, lse, do, seg, w.head_kind, w.scale)
    torch.cuda.synchronize()
    sum_do = (do.float() * nonpad).sum(dim=2)                 # [B, H, D]
    sum_dv = dv.float().sum(dim=2)
    n_tok = nonpad.sum(dim=2).clamp(min=1).float()            # rounding of n_tok bf16 values
    # bf16 rounding of n_tok values: observed 2e-3; one missing 128-row unit would give ~1e-1
    assert float(((sum_dv - sum_do).abs() / n_tok.sqrt()).max()) <= 8e-3
    sum_dk = dk.float().sum(dim=2)
    scale_k = dk.float().abs().sum(dim=2).clamp(min=1e-3)
    assert float((sum_dk.abs() / scale_k).max()) <= 8e-3      # observed 4e-4 .. 2e-3
    assert bool(torch.isfinite(dq.float()).all())


def test_backward_is_bit_reproducible():
    from paper_2109_04312_amd import mate
    w = small_workload(5, "bf16", B=2, N=700, H=4, max_rows=40, max_cols=6, max_global=70, max_cell=5)
    r, c, f = hp.dev_structure(w.structure)
    seg = mate.build_segments(r, c, f)
    q, k, v, do = (hp.to_dev(x, "bf16") for x in (w.q, w.k, w.v, w.do))
    out, lse = mate.attn_fwd(q, k, v, seg, w.head_kind, w.scale)
    a = mate.attn_bwd(q, k, v, out, lse, do, seg, w.head_kind, w.scale)
    b = mate.attn_bwd(q, k, v, out, lse, do, seg, w.head_kind, w.scale)
    out2, lse2 = mate.attn_fwd(q, k, v, seg, w.head_kind, w.scale)
    torch.cuda.synchronize()
    for x, y in zip(a, b):
        assert torch.equal(x, y)
    assert torch.equal(out, out2) and torch.equal(lse, lse2)


@pytest.mark.parametrize("id_step,N,rows,cols", [(1, 4096, 30, 15), (1000, 4096, 30, 15), (1, 8192, 62, 31)])
def test_more_unit_cuts_than_records(id_step, N, rows, cols):
    """Every row is a segment of 129 slots and every column one of 258: cutting at each of them
    would need more unit records than a view has, so the builder falls back to a cut every 128 slots,
    and units straddle long segments again.  Each way to list units: one wavefront (up to 64
    records), the workgroup (8192 positions have 98), and id_step = 1000, which takes the ids past the
    counting sort's range (general sorting path)."""
    L, G, P = synth.TOK_LOCAL, synth.TOK_GLOBAL, synth.TOK_PAD
    flags = np.full((1, N), P, np.uint8)
    row = np.zeros((1, N), np.int32)
    col = np.zeros((1, N), np.int32)
    flags[0, :20] = G
    n = rows * 129
    assert n == cols * 258 and 20 + n <= N
    flags[0, 20:20 + n] = L
    i = np.arange(n)
    row[0, 20:20 + n] = (1 + i // 129) * id_step
    col[0, 20:20 + n] = (1 + i % cols) * id_step
    st = synth.Structure(row, col, flags)
    rng = np.random.default_rng(129 + id_step)
    q, k, v, do = synth.draw_tensors(rng, 1, 2, N, 64, "bf16", 4)
    w = synth.Workload(f"cuts_step{id_step}_{N}", "bf16", st, np.array([ROW, COL], np.uint8), q, k, v, do, 0.125)
    check_workload(w, backward=True)


@pytest.mark.parametrize("segments,N", [(63, 500), (64, 500), (65, 700), (128, 700), (129, 700), (128, 2000), (100, 5248), (100, 5249)])
def test_units_of_as_many_segments_as_lanes(segments, N):
    """Work units listed by one wavefront (a segment or two to a lane) and by all: segment counts beside 64 and 128, and 63
    and 65 records (5248 and 5249 positions), with a long segment among short ones in each view."""
    rng = np.random.default_rng(segments + N)
    ids = np.sort(np.concatenate([np.arange(segments), rng.integers(0, segments, N - segments)]))
    row = np.stack([np.where(rng.random(N) < 0.4, segments // 2, ids), rng.permutation(ids)]).astype(np.int32)
    col = np.stack([rng.permutation(ids), np.where(rng.random(N) < 0.3, 0, ids)]).astype(np.int32)
    flags = (rng.random((2, N)) < 0.05).astype(np.uint8)
    flags[1, N - 40:] = synth.TOK_PAD
    q, k, v, do = synth.draw_tensors(rng, 2, 2, N, 64, "bf16", 4)
    w = synth.Workload(f"lanes{segments}", "bf16", synth.Structure(row, col, flags), np.array([ROW, COL], np.uint8), q, k, v, do, 0.125)
    check_workload(w, backward=True)


@pytest.mark.parametrize("B,N,H", [(187, 60, 16), (188, 60, 16), (2, 1999, 256), (20, 700, 40)])
def test_launches_on_either_side_of_many_records(B, N, H):
    """12000 records: a unit is found in one round trip below, step by step above (chunks joined: 2 x 1999 with 256 heads)."""
    w = small_workload(N, "bf16", B=B, N=N, H=H, max_rows=30, max_cols=6, max_global=min(N // 4, 40))
    check_workload(w, backward=True, pairs=[(0, 0), (0, H - 1), (B // 2, 1), (B - 1, H - 2), (B - 1, H - 1)])


# small launches on either side of where units are found step by step: the backward of one or two tiles from 1152 workgroups on (8 and
# 9 sequences of 60 with 16 heads, 5 and 6 of 200; three tiles never), the forward of one tile from 640 records on (9 and 10
# of 60; 10 of 128 with a result beyond 2 MB), the f32 backward beyond 20000 workgroups
@pytest.mark.parametrize("dtype,B,N,H", [("bf16", 8, 60, 16), ("bf16", 9, 60, 16), ("bf16", 10, 60, 16), ("bf16", 10, 128, 16), ("bf16", 5, 200, 16),
                                         ("bf16", 6, 200, 16), ("bf16", 5, 300, 16), ("f32", 22, 130, 16), ("f32", 23, 130, 16)])
def test_small_launches_on_either_side_of_many_records(dtype, B, N, H):
    w = small_workload(N, dtype, B=B, N=N, H=H, max_rows=12, max_cols=6, max_global=min(N // 4, 40))
    check_workload(w, backward=True, pairs=[(0, 0), (0, H - 1), (B // 2, 1), (B - 1, H - 2), (B - 1, H - 1)])


@pytest.mark.parametrize("dtype,B,N", [("bf16", 4, 341), ("bf16", 4, 342), ("f32", 2, 341), ("f32", 2, 342)])
def test_results_on_either_side_of_two_megabytes(dtype, B, N):
    """A small forward's result stays in the L2 or passes through it (12 heads: 341 positions are the last below 2 MB)."""
    check_workload(small_workload(N, dtype, B=B, N=N, H=12, bwd=False, max_rows=30, max_cols=6, max_global=20), backward=False)


def test_head_kind_mix_and_order():
    # any assignment of kinds to heads, not only "first half rows"
    w = small_workload(8, "bf16", B=1, N=260, H=5, max_rows=10, max_cols=5, max_global=9)
    w.head_kind = np.array([COL, COL, ROW, COL, ROW], np.uint8)
    check_workload(w, backward=True)


@pytest.mark.parametrize("kinds", [(ROW, ROW, ROW), (COL, COL, COL), (ROW, COL, COL)])
def test_single_kind_and_odd_pair_counts(kinds):
    # only row heads / only column heads; B * H = 9 is not a multiple of the eight work queues
    w = small_workload(11, "bf16", B=3, N=300, H=3, max_rows=12, max_cols=5, max_global=20)
    w.head_kind = np.array(kinds, np.uint8)
    check_workload(w, backward=True, label=f"kinds{kinds}")


def test_argument_errors_leave_outputs_untouched():
    from paper_2109_04312_amd import mate
    w = small_workload(1, "f32", B=1, N=64, H=2, bwd=False)
    r, c, f = hp.dev_structure(w.structure)
    seg = mate.build_segments(r, c, f)
    q = hp.to_dev(w.q, "f32")
    out = torch.full_like(q, 7.0)
    lse = torch.full((1, 2, 64), 7.0, device="cuda")
    hk = np.array([0, 9], np.uint8)
    st = mate.mate_attn_fwd(q.data_ptr(), q.data_ptr(), q.data_ptr(), seg.buf.data_ptr(), hk.ctypes.data,
                            1, 2, 64, 64, 0, 0.125, out.data_ptr(), lse.data_ptr(), None, 0, None)
    assert st == mate.MATE_ERR_UNSUPPORTED
    torch.cuda.synchronize()
    assert bool((out == 7).all()) and bool((lse == 7).all())


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_tables_of_another_shape_leave_outputs_untouched(dtype):
    """The attention calls are asynchronous and cannot return what only the device sees: given a
    table buffer that was built for another (B, N), or never built, every workgroup leaves before
    using it, the outputs stay as they were, and mate_segments_status names the problem."""
    from paper_2109_04312_amd import mate
    w = small_workload(31, dtype, B=2, N=300, H=2, max_rows=9, max_cols=4, max_global=12)
    r, c, f = hp.dev_structure(w.structure)
    q, k, v, do = (hp.to_dev(x, dtype) for x in (w.q, w.k, w.v, w.do))
    B, H, N, D = q.shape
    code = mate.MATE_BF16 if dtype == "bf16" else mate.MATE_F32
    hk = np.ascontiguousarray(w.head_kind)
    nbytes = max(mate.mate_segments_bytes(B, N), mate.mate_segments_bytes(1, 200))
    other = mate.Segments(torch.zeros(nbytes, dtype=torch.uint8, device="cuda"), 1, 200)
    mate.build_segments(r[:1, :200].contiguous(), c[:1, :200].contiguous(), f[:1, :200].contiguous(), out=other)
    never = torch.full((nbytes,), 0x5A, dtype=torch.uint8, device="cuda")
    good = mate.build_segments(r, c, f)
    assert mate.segments_status(good) == mate.MATE_OK
    assert mate.mate_segments_status(other.buf.data_ptr(), B, N, None) == mate.MATE_ERR_SHAPE
    assert mate.mate_segments_status(never.data_ptr(), B, N, None) == mate.MATE_ERR_SHAPE
    out_ref, lse_ref = mate.attn_fwd(q, k, v, good, hk, 0.125)
    ws_f = mate.workspace(B, H, N, D, code, False, "cuda")
    ws_b = mate.workspace(B, H, N, D, code, True, "cuda")
    for buf in (other.buf, never):
        out = torch.full_like(q, 7.0)
        lse = torch.full((B, H, N), 7.0, device="cuda")
        grads = [torch.full_like(q, 7.0) for _ in range(3)]
        st = mate.mate_attn_fwd(q.data_ptr(), k.data_ptr(), v.data_ptr(), buf.data_ptr(), hk.ctypes.data,
                                B, H, N, D, code, 0.125, out.data_ptr(), lse.data_ptr(),
                                ws_f.data_ptr(), ws_f.numel(), None)
        assert st == mate.MATE_OK          # nothing the host can see is wrong
        st = mate.mate_attn_bwd(q.data_ptr(), k.data_ptr(), v.data_ptr(), out_ref.data_ptr(), lse_ref.data_ptr(),
                                do.data_ptr(), buf.data_ptr(), hk.ctypes.data, B, H, N, D, code, 0.125,
                                *(g.data_ptr() for g in grads), ws_b.data_ptr(), ws_b.numel(), None)
        assert st == mate.MATE_OK
        torch.cuda.synchronize()
        for t in (out, lse, *grads):
            assert bool((t == 7).all())
    with pytest.raises(mate.MateError) as e:      # the binding knows the shape its tables were built for
        mate.attn_fwd(q, k, v, other, hk, 0.125)
    assert e.value.status == mate.MATE_ERR_SHAPE


def test_invalid_ids_are_reported_by_the_status_call():
    from paper_2109_04312_amd import mate
    w = small_workload(32, "bf16", B=3, N=150, H=2, max_rows=6, max_cols=4, max_global=5)
    st = w.structure
    table = np.flatnonzero(st.flags[1] == synth.TOK_LOCAL)
    st.row_ids[1, table[3]] = -4                     # a negative id on a table token of sequence 1
    r, c, f = hp.dev_structure(st)
    seg = mate.build_segments(r, c, f)
    assert mate.segments_status(seg) == mate.MATE_ERR_BAD_ID
    # the tables are still consistent, so the attention runs and writes every row
    q, k, v = (hp.to_dev(x, "bf16") for x in (w.q, w.k, w.v))
    out, lse = mate.attn_fwd(q, k, v, seg, w.head_kind, 0.125, out=torch.full_like(q, float("nan")))
    torch.cuda.synchronize()
    assert bool(torch.isfinite(out).all())
    st.row_ids[1, table[3]] = 0
    st.flags[2, 5] = 9                               # a flag value above 2
    r, c, f = hp.dev_structure(st)
    assert mate.segments_status(mate.build_segments(r, c, f)) == mate.MATE_ERR_BAD_ID


def test_step_replays_identically_from_a_captured_graph():
    """The library allocates nothing, clears nothing with memsets and never synchronises inside
    build / forward / backward, so a whole step can be captured once and replayed: every replay
    (with eager work in between) must reproduce the eager result bit for bit."""
    from paper_2109_04312_amd import mate
    w = small_workload(21, "bf16", B=2, N=900, H=4, max_rows=30, max_cols=6, max_global=80, max_cell=6)
    r, c, f = hp.dev_structure(w.structure)
    q, k, v, do = (hp.to_dev(x, "bf16") for x in (w.q, w.k, w.v, w.do))
    B, H, N, D = q.shape
    code = mate.MATE_BF16

    def buffers():
        seg = mate.Segments(torch.zeros(mate.mate_segments_bytes(B, N), dtype=torch.uint8, device="cuda"), B, N)
        return dict(seg=seg, out=torch.empty_like(q), lse=torch.empty((B, H, N), dtype=torch.float32, device="cuda"),
                    dq=torch.empty_like(q), dk=torch.empty_like(q), dv=torch.empty_like(q),
                    ws_f=mate.workspace(B, H, N, D, code, False, "cuda"), ws_b=mate.workspace(B, H, N, D, code, True, "cuda"))

    def step(bf):
        mate.build_segments(r, c, f, out=bf["seg"])
        mate.attn_fwd(q, k, v, bf["seg"], w.head_kind, w.scale, out=bf["out"], lse=bf["lse"], ws=bf["ws_f"])
        mate.attn_bwd(q, k, v, bf["out"], bf["lse"], do, bf["seg"], w.head_kind, w.scale,
                      dq=bf["dq"], dk=bf["dk"], dv=bf["dv"], ws=bf["ws_b"])

    eager, graphed = buffers(), buffers()
    step(eager)
    torch.cuda.synchronize()
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        step(graphed)                                  # warm-up on the capture stream
    torch.cuda.current_stream().wait_stream(side)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=side):
        step(graphed)
    for replay in range(3):
        for name in ("out", "lse", "dq", "dk", "dv"):
            graphed[name].fill_(float("nan"))          # a replay must rewrite everything
        step(eager)                                     # eager work between the replays
        graph.replay()
        torch.cuda.synchronize()
        for name in ("out", "lse", "dq", "dk", "dv"):
            assert torch.equal(graphed[name], eager[name]), (replay, name)


@pytest.mark.parametrize("n_global,rows,cols,cell,N", [(31, 3, 1, 32, 127), (32, 2, 2, 32, 161), (33, 1, 3, 33, 132),
                                                       (1, 1, 1, 1, 2), (65, 31, 2, 3, 260), (40, 90, 5, 4, 2100)])
def test_f32_tile_edges(n_global, rows, cols, cell, N):
    """Lists and segments at and beside multiples of the 32-row tiles; the last one is long enough for
    question-token owners that the tables cut into chunks."""
    st = synth._stack([synth.flatten_table(N, n_global, rows, cols, np.full(rows * cols, cell))])
    q, k, v, do = synth.draw_tensors(np.random.default_rng(N), 1, 2, N, 64, "f32", 4)
    check_workload(synth.Workload(f"f32 edges {N}", "f32", st, np.array([ROW, COL], np.uint8), q, k, v, do, 0.125), True)


@pytest.mark.parametrize("B,N,H,n_global", [(42, 300, 2, 40), (43, 300, 2, 40), (65, 120, 2, 3), (16, 500, 2, 33), (17, 500, 2, 33), (4, 2100, 2, 140)])
def test_f32_forward_in_either_order_of_units(B, N, H, n_global):
    """A launch of more than 128 tiles of owners (B H ceil(N / 128): 130, 128, 136 and 136 in the last four) starts its question-token
    owners before the columns', with two or three tiles a sequence one of more than 256 (252 and 258); a smaller one after them."""
    w = chunked_workload(N, B, N, H, n_global, "f32")
    got, _ = hp.run_hip(w, False)
    print(hp.report(hp.compare(got, hp.run_oracle(w, False, [(b, h) for b in (0, B - 1) for h in range(H)]), w, w.name)), flush=True)


@pytest.mark.parametrize("B,N,H,n_global", [(2, 384, 12, 40), (2, 385, 8, 40), (2, 385, 10, 40), (1, 700, 12, 130), (1, 1100, 12, 70)])
def test_f32_backward_in_either_order_of_units(B, N, H, n_global):
    """Owners of question tokens after the column heads' units and before them: three tiles of owners and four, 64 tiles
    a launch and 80, and sequences with two tiles of question tokens."""
    w = chunked_workload(N, B, N, H, n_global, "f32")
    check_workload(w, True, pairs=[(0, 0), (0, H - 1), (B - 1, 1), (B - 1, H - 1)])


@pytest.mark.parametrize("rise", [0, 12])
@pytest.mark.parametrize("n_global,rows,cols,cell,N", [(1, 1, 1, 1, 2), (31, 3, 1, 32, 127), (32, 5, 2, 13, 170),
                                                       (33, 4, 3, 33, 440), (64, 2, 2, 65, 330), (65, 31, 2, 3, 260),
                                                       (40, 90, 5, 4, 2100), (96, 3, 2, 200, 1300)])
def test_bf16_tile_edges(n_global, rows, cols, cell, N, rise):
    """Lists and segments at and beside multiples of the 32-row blocks, units of more and of at most 64 rows;
    with `rise` (forward only) the scores grow along the sequence: later tiles need a new softmax reference."""
    st = synth._stack([synth.flatten_table(N, n_global, rows, cols, np.full(rows * cols, cell))])
    q, k, v, do = synth.draw_tensors(np.random.default_rng(N), 1, 2, N, 64, "bf16", 4)
    k = synth.round_to_bf16(k * (1 + rise * np.arange(N, dtype=np.float32)[:, None] / N))
    check_workload(synth.Workload(f"bf16 edges {N}", "bf16", st, np.array([ROW, COL], np.uint8), q, k, v, do, 0.125), rise == 0)


@pytest.mark.parametrize("n_global,columns,N", [(3, 40, 823), (37, 40, 900), (64, 23, 340)])
def test_windows_of_every_length_at_every_offset(n_global, columns, N):
    """Columns of 1, 2, 3, ... tokens: windows that begin and end at every place in the eight rows of a block that a lane masks."""
    st = synth._stack([synth.flatten_table(N, n_global, 1, columns, np.arange(1, columns + 1))])
    q, k, v, do = synth.draw_tensors(np.random.default_rng(N), 1, 2, N, 64, "bf16", 4)
    check_workload(synth.Workload(f"columns of 1 to {columns}", "bf16", st, np.array([ROW, COL], np.uint8), q, k, v, do, 0.125), True)


@pytest.mark.parametrize("bits", [12, 14, 50, 95, 110, 140])
@pytest.mark.parametrize("n_global,rows,cols,cell,N", [(31, 3, 2, 40, 271), (70, 2, 3, 100, 670), (40, 90, 5, 4, 2100)])
def test_bf16_scores_that_rise_in_steps(n_global, rows, cols, cell, N, bits):
    """Every fifth of the sequence scores 2^bits more than the one before: below 2^13 per tile the softmax reference
    stays, above it the tile is done again and the reference follows the maximum from there on."""
    st = synth._stack([synth.flatten_table(N, n_global, rows, cols, np.full(rows * cols, cell))])
    rng = np.random.default_rng(bits)
    q, k, v = synth.draw_tensors(rng, 1, 2, N, 64, "bf16", 3)
    u = np.full(64, 0.125, np.float32)
    step = np.arange(N, dtype=np.float32) * 5 // N
    q = synth.round_to_bf16(0.3 * q + 16.0 * u)
    k = synth.round_to_bf16(0.3 * k + (step * bits * np.log(2) / (0.125 * 16.0))[:, None] * u)
    w = synth.Workload(f"steps{bits}_{N}", "bf16", st, np.array([ROW, COL], np.uint8), q, k, v, None, 0.125)
    check_workload(w, backward=False)
    if N <= 1024:
        print(hp.report(hp.compare(hp.run_hip(w, False, dense=True)[0], hp.run_oracle(w, False), w, "dense steps")))


@pytest.mark.parametrize("n_global,table,N,H", [(60, 700, 768, 120),     # 12 tiles: two chunks, joined a whole stream
                                                (20, 790, 832, 104),     # 14: three
                                                (40, 1060, 1100, 80),    # 18: three
                                                (130, 1370, 1500, 64),   # 25, two owner tiles of question tokens
                                                (64, 2490, 2560, 36),    # 40: four
                                                (64, 2500, 2600, 36)])   # 41: as the tables list them
def test_chunks_in_pairs_where_many_heads_fill_the_chip(n_global, table, N, H):
    """Small batches with many heads run the short chunks of question-token owners in pairs.  All row heads have the same
    inputs and so have all column heads; one of each is compared with the oracle, the others with it."""
    cols, cell = 5, 10
    cells = table // cell
    st = synth._stack([synth.flatten_table(N, n_global, cells // cols, cols, np.full(cells // cols * cols, cell))])
    hk = synth.half_row_half_col(H)
    pair = synth.draw_tensors(np.random.default_rng(N), 1, 2, N, 64, "bf16", 4)
    w = synth.Workload(f"pairs {N}", "bf16", st, hk, *(np.ascontiguousarray(x[:, hk]) for x in pair), 0.125)
    got, _ = hp.run_hip(w, True)
    first = {int(kind): int(np.argmax(hk == kind)) for kind in (ROW, COL)}
    print(hp.report(hp.compare(got, hp.run_oracle(w, True, [(0, h) for h in first.values()]), w, w.name)), flush=True)
    for name, x in got.items():
        for h in range(H):
            assert np.array_equal(x[0, h], x[0, first[int(hk[h])]]), (name, h)


# a joined stream; two owner tiles of question tokens; a stream so long that its chunks are not joined
@pytest.mark.parametrize("n_global,table,N,few,many", [(60, 950, 1024, 96, 128), (130, 1370, 1500, 64, 80), (64, 2500, 2600, 36, 40)])
def test_chunks_in_pairs_with_gradients_at_once_and_one_after_the_other(n_global, table, N, few, many):
    """Up to 768 units (heads times ceil(N / 128); `few` heads have 768 or 756, `many` 1024, 960 and 840) dQ and dK/dV are one
    launch and dQ's chunks are merged by the last to arrive, beyond by the first workgroups of dK/dV's launch: the same bits.
    Heads of a kind have the same inputs."""
    cols, cell = 5, 10
    cells = table // cell
    st = synth._stack([synth.flatten_table(N, n_global, cells // cols, cols, np.full(cells // cols * cols, cell))])
    pair = synth.draw_tensors(np.random.default_rng(N), 1, 2, N, 64, "bf16", 4)
    first = {}
    for H in (few, many):
        hk = synth.half_row_half_col(H)
        w = synth.Workload(f"pairs {N} {H}", "bf16", st, hk, *(np.ascontiguousarray(x[:, hk]) for x in pair), 0.125)
        got, _ = hp.run_hip(w, True)
        at = {int(kind): int(np.argmax(hk == kind)) for kind in (ROW, COL)}
        first = first or {(name, kind): x[0, h] for name, x in got.items() for kind, h in at.items()}
        for name, x in got.items():
            for h in range(H):
                assert np.array_equal(x[0, h], first[name, int(hk[h])]), (name, H, h)
    print(hp.report(hp.compare(got, hp.run_oracle(w, True, [(0, h) for h in at.values()]), w, w.name)), flush=True)


def chunked_workload(seed, B, N, H, n_global=80, dtype="bf16"):
    """Sequences filled to the last position, whose question-token owners' streams are cut into several chunks."""
    rng = np.random.default_rng(seed)
    cols, cell = 6, 5
    rows = -(-N // (cols * cell))
    st = synth._stack([synth.flatten_table(N, n_global, rows, cols, np.full(rows * cols, cell)) for _ in range(B)])
    hk = synth.half_row_half_col(H)
    return synth.Workload(f"chunks{seed}", dtype, st, hk, *synth.draw_tensors(rng, B, H, N, 64, dtype, 4), 0.125)


def arrival_words(ws, B, H, N):
    """The arrival words at the end of a workspace: one per question-token unit that a sequence can have."""
    return ws.view(torch.int64)[-B * H * ((N + 127) // 128):].view(B * H, -1)


# Chunks of 16 tiles (B N > 4096), short ones, short ones in pairs, and two owner tiles of question tokens.  Units (B H
# ceil(N / 128)) 136, 68, 768 and 32: dQ and dK/dV in one launch; the forward is fwd_small_kernel up to 512 (with question-token
# owners of more than 32 rows, one tile at a time), fwd_mfma_kernel<., true> at 768.  Then, in this order: owners of at most
# 32 rows, two tiles at a time (48 units); short chunks on fwd_mfma_kernel<true, false>, still one backward launch (576); chunks
# of 16 tiles there, with dQ and dK/dV one after the other, dQ's chunks merged by dK/dV's first workgroups (1280); short
# ones in pairs and one after the other (960).
CHUNKED = [(2, 2100, 4, 80), (1, 2100, 4, 80), (1, 1500, 64, 40), (1, 2000, 2, 200),
           (1, 1500, 4, 20), (1, 2000, 36, 60), (2, 5000, 16, 140), (1, 1500, 80, 40)]


@pytest.mark.parametrize("B,N,H,n_global", CHUNKED)
def test_chunked_owners_are_bit_reproducible_whatever_the_workspace_held(B, N, H, n_global):
    """Which chunk merges depends on the run; what it computes does not.  The forward's words are cleared when it is
    done, all of a group's or none; the backward's first word of a group has counted the group's chunks."""
    from paper_2109_04312_amd import mate
    w = chunked_workload(N + B, B, N, H, n_global)
    ids = hp.dev_structure(w.structure)
    seg = mate.build_segments(*ids)
    q, k, v, do = (hp.to_dev(x, "bf16") for x in (w.q, w.k, w.v, w.do))
    ws_f, ws_b = (mate.workspace(B, H, N, 64, mate.MATE_BF16, back, "cuda") for back in (False, True))
    first = None
    for garbage in (0, 0x5A, 0xFF, 0, 0x5A, 0xFF):
        ws_f.fill_(garbage)
        ws_b.fill_(garbage)
        out, lse = mate.attn_fwd(q, k, v, seg, w.head_kind, w.scale, ws=ws_f)
        res = (out, lse, *mate.attn_bwd(q, k, v, out, lse, do, seg, w.head_kind, w.scale, ws=ws_b))
        first = first or res
        for name, x, y in zip(("out", "lse", "dq", "dk", "dv"), res, first):
            assert torch.equal(x, y), (name, garbage)
        if garbage:
            cleared = (arrival_words(ws_f, B, H, N) == 0).sum(1)
            counted = arrival_words(ws_b, B, H, N)
            counted = torch.where((counted > 0) & (counted < 256), counted, 0).sum(1)
            print("chunks per (sequence, head):", cleared.unique().tolist(), flush=True)
            assert bool((cleared > 1).all()) and torch.equal(cleared, counted)


@pytest.mark.parametrize("B,N,H,n_global", CHUNKED)
def test_chunked_owners_replay_identically_from_a_captured_graph(B, N, H, n_global):
    """A captured forward keeps its ticket: its words must be cleared for the next replay, also when other calls
    have used the same workspace in between."""
    from paper_2109_04312_amd import mate
    w = chunked_workload(N - B, B, N, H, n_global)
    r, c, f = hp.dev_structure(w.structure)
    q, k, v, do = (hp.to_dev(x, "bf16") for x in (w.q, w.k, w.v, w.do))
    seg = mate.Segments(torch.zeros(mate.mate_segments_bytes(B, N), dtype=torch.uint8, device="cuda"), B, N)
    res = dict(out=torch.empty_like(q), lse=torch.empty((B, H, N), dtype=torch.float32, device="cuda"),
               dq=torch.empty_like(q), dk=torch.empty_like(q), dv=torch.empty_like(q))
    ws_f, ws_b = (mate.workspace(B, H, N, 64, mate.MATE_BF16, back, "cuda") for back in (False, True))

    def step():
        mate.build_segments(r, c, f, out=seg)
        mate.attn_fwd(q, k, v, seg, w.head_kind, w.scale, out=res["out"], lse=res["lse"], ws=ws_f)
        mate.attn_bwd(q, k, v, res["out"], res["lse"], do, seg, w.head_kind, w.scale,
                      dq=res["dq"], dk=res["dk"], dv=res["dv"], ws=ws_b)

    side = torch.cuda.Stream()
    with torch.cuda.stream(side):
        step()
    torch.cuda.synchronize()
    want = {n: x.clone() for n, x in res.items()}
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=side):
        step()
    for replay in range(6):
        if replay % 2:
            step()                       # an eager call on the same buffers
            torch.cuda.synchronize()
        for x in res.values():
            x.fill_(float("nan"))
        graph.replay()
        torch.cuda.synchronize()
        for n, x in res.items():
            assert torch.equal(x, want[n]), (replay, n)


def pairwise_reference(w, bad):
    """Forward and backward in float64 from explicit key and query lists, so that a value of a token reaches exactly
    the tokens that meet it (a masked matrix product would multiply it with zeros).  {(b, h): dict}, on tensors
    `bad` = (q, k, v, do)."""
    st, ref = w.structure, {}
    for b in range(st.B):
        for h, kind in enumerate(w.head_kind):
            meets = orc.attention_mask(st.row_ids[b], st.col_ids[b], st.flags[b], int(kind)).astype(bool)
            q, k, v, do = (x[b, h].astype(np.float64) for x in bad)
            d = {n: np.zeros_like(q) for n in ("o", "dq", "dk", "dv")}
            d["lse"] = np.zeros(len(q))
            p, ds = np.zeros(meets.shape), np.zeros(meets.shape)
            for i in np.flatnonzero(meets.any(1)):
                keys = np.flatnonzero(meets[i])
                s = w.scale * (k[keys] @ q[i])
                mx = s.max()
                e = np.exp(s - mx)
                d["o"][i] = (e / e.sum()) @ v[keys]
                d["lse"][i] = mx + np.log(e.sum())
                p[i, keys] = np.exp(s - d["lse"][i])
                ds[i, keys] = p[i, keys] * (v[keys] @ do[i] - do[i] @ d["o"][i])
                d["dq"][i] = w.scale * (ds[i, keys] @ k[keys])
            for j in np.flatnonzero(meets.any(0)):
                rows = np.flatnonzero(meets[:, j])
                d["dk"][j] = w.scale * (ds[rows, j] @ q[rows])
                d["dv"][j] = p[rows, j] @ do[rows]
            ref[(b, h)] = d
    return ref


@pytest.mark.parametrize("value", [float("inf"), float("nan")])
@pytest.mark.parametrize("tensor", ["q", "k", "v", "do"])
@pytest.mark.parametrize("whole_row", [False, True])
def test_f32_special_values_reach_only_the_tokens_that_meet_them(tensor, value, whole_row):
    """An Inf or NaN in one row of an input: outputs are non-finite exactly where the definition makes them so, and
    right everywhere else.  The table token is the last of its row and column (tiles repeat the last one)."""
    from paper_2109_04312_amd import mate
    n_global, rows, cols, cell, N = 33, 9, 5, 4, 230
    st = synth._stack([synth.flatten_table(N, n_global, rows, cols, np.full(rows * cols, cell))])
    t = dict(zip(("q", "k", "v", "do"), synth.draw_tensors(np.random.default_rng(3), 1, 2, N, 64, "f32", 4)))
    w = synth.Workload("special", "f32", st, np.array([ROW, COL], np.uint8), *t.values(), 0.125)
    at = n_global + rows * cols * cell - 1
    assert st.flags[0, at] == synth.TOK_LOCAL and st.flags[0, at + 1] == synth.TOK_PAD
    t[tensor][0, :, at, slice(None) if whole_row else 17] = value
    with np.errstate(all="ignore"):
        ref = pairwise_reference(w, t.values())
    ids = hp.dev_structure(st)
    q, k, v, do = (hp.to_dev(x, "f32") for x in t.values())
    seg = mate.build_segments(*ids)
    out, lse = mate.attn_fwd(q, k, v, seg, w.head_kind, w.scale)
    got = dict(zip(("o", "lse", "dq", "dk", "dv"), (out, lse, *mate.attn_bwd(q, k, v, out, lse, do, seg, w.head_kind, w.scale))))
    for (b, h), d in ref.items():
        for name, r in d.items():
            g = got[name][b, h].double().cpu().numpy()
            fine = np.isfinite(r)
            print(tensor, value, h, name, "finite", int(fine.sum()), "of", fine.size, flush=True)
            assert np.array_equal(np.isfinite(g), fine), (name, h)
            assert np.abs(g[fine] - r[fine]).max(initial=0.0) <= 1e-4, (name, h)


@pytest.mark.parametrize("B,N,H,n_global", [(2, 5000, 16, 140), (22, 300, 12, 40)])
def test_backward_of_a_batch_in_parts(B, N, H, n_global):
    """A large launch runs dQ and dK/dV one after the other, a small one both at once (B H ceil(N / 128) of 1280 and 640,
    792 and 396 units, with chunks of question-token owners and without): the same bits."""
    from paper_2109_04312_amd import mate
    w = chunked_workload(N, B, N, H, n_global)
    r, c, f = hp.dev_structure(w.structure)
    q, k, v, do = (hp.to_dev(x, "bf16") for x in (w.q, w.k, w.v, w.do))
    out, lse = mate.attn_fwd(q, k, v, mate.build_segments(r, c, f), w.head_kind, w.scale)
    whole = mate.attn_bwd(q, k, v, out, lse, do, mate.build_segments(r, c, f), w.head_kind, w.scale)
    for part in (slice(0, B // 2), slice(B // 2, B)):
        seg = mate.build_segments(*(x[part].contiguous() for x in (r, c, f)))
        some = mate.attn_bwd(*(x[part].contiguous() for x in (q, k, v, out, lse, do)), seg, w.head_kind, w.scale)
        torch.cuda.synchronize()
        for name, x, y in zip(("dq", "dk", "dv"), some, whole):
            assert torch.equal(x, y[part]), (part, name)


@pytest.mark.parametrize("values", ["ordinary", "wide", "no split", "small q", "small k", "small v", "small do",
                                    "small products", "small probabilities", "zeros", "zero v", "small v that cancels"])
def test_f32_products_from_splits(values):
    """fp32 products are formed from three bf16 parts: as good as fp32 over 120 binary orders of magnitude, for a value
    above the largest bf16, which has no such parts, and for values whose parts would not be normal numbers (an input, or
    P and dS, of 2^-120 keeps 14 bits in parts of bf16, none below 2^-126).  Bounds: a product and its share of an fp32 sum
    are within a few 2^-24 of their size, P within 2^-24 times the exponents of a score of a few units, of its own; where
    scores spread by 82 (118 in base 2), a score and the log-sum-exp are within a few 2^-18, and with them P."""
    from paper_2109_04312_amd import mate
    n_global, rows, cols, cell, N = 33, 9, 5, 4, 230
    st = synth._stack([synth.flatten_table(N, n_global, rows, cols, np.full(rows * cols, cell))])
    rng = np.random.default_rng(4)
    q, k, v, do = synth.draw_tensors(rng, 1, 2, N, 64, "f32", 4)
    at = n_global + rows * cols * cell - 1
    if values == "wide":
        v, do = (x * np.exp2(rng.integers(-60, 61, (1, 2, N, 1))).astype(np.float32) for x in (v, do))
    elif values == "no split":
        v[0, :, at], do = np.float32(3.4e38), do * np.float32(2.0 ** -40)
    elif values in ("small q", "small k"):       # (scores are as ever)
        sign = -1 if values == "small q" else 1
        q, k = q * np.float32(2.0 ** (120 * sign)), k * np.float32(2.0 ** (-120 * sign))
    elif values == "small v":
        v = v * np.float32(2.0 ** -120)
    elif values == "small do":
        do = do * np.float32(2.0 ** -120)
    elif values == "small products":             # dP and dS
        v, do = v * np.float32(2.0 ** -60), do * np.float32(2.0 ** -60)
    elif values == "small probabilities":        # some keys take it all and have nothing to give
        q, k = q * np.float32(0.3), k * np.float32(0.3)
        q[..., 0], k[..., 0] = 32, 0
        k[:, :, ::5, 0], v[:, :, ::5] = 20.5, 0
    elif values == "zeros":
        v[..., ::3], do[:, :, ::2], k[:, :, 40:80], q[..., 5] = 0, 0, 0, 0
    elif values == "zero v":
        v[:] = 0
    elif values == "small v that cancels":       # out of O and delta, not out of dP and dK: 16 bits, the last at 2^-135
        k[:] = 0
        v[:] = (2.0 ** -120 * (1 + 2.0 ** -15) * (1 - 2 * (np.arange(N) % 2)))[:, None]
        v[:, :, n_global - 2] *= 2
        do = do * np.float32(2.0 ** 60)
    w = synth.Workload("splits", "f32", st, np.array([ROW, COL], np.uint8), q, k, v, do, 0.125)
    ref = pairwise_reference(w, (q, k, v, do))
    dev = [hp.to_dev(x, "f32") for x in (q, k, v, do)]
    seg = mate.build_segments(*hp.dev_structure(st))
    out, lse = mate.attn_fwd(*dev[:3], seg, w.head_kind, w.scale)
    got = dict(zip(("o", "dq", "dk", "dv"), (out, *mate.attn_bwd(*dev[:3], out, lse, dev[3], seg, w.head_kind, w.scale))))
    for (b, h), d in ref.items():
        Q, K, V, G = (x[b, h].astype(np.float64) for x in (q, k, v, do))
        meets = orc.attention_mask(st.row_ids[b], st.col_ids[b], st.flags[b], int(w.head_kind[h])).astype(bool)
        p = np.where(meets, np.exp(w.scale * (Q @ K.T) - d["lse"][:, None]), 0.0)
        ds = p * (np.abs(G) @ np.abs(V).T + (np.abs(G) * np.abs(d["o"])).sum(1)[:, None])
        size = {"o": p @ np.abs(V), "dv": p.T @ np.abs(G), "dq": w.scale * ds @ np.abs(K), "dk": w.scale * ds.T @ np.abs(Q)}
        for name, s in size.items():
            ratio = np.abs(got[name][b, h].double().cpu().numpy() - d[name]) / np.maximum(s, 1e-300)
            print(values, h, name, "max error %.1e of its size" % ratio.max(), flush=True)
            assert ratio.max() <= (512 if values == "small probabilities" else 32) * 2.0 ** -24, (name, h)


@pytest.mark.parametrize("n_global,N", [(1, 130), (32, 160), (32, 200), (31, 321), (33, 321), (32, 700), (7, 1500)])
def test_owners_that_all_wavefronts_meet_two_tiles_at_a_time(n_global, N):
    """Small launches, question-token owners of at most 32 rows: three, an odd and an even number of tiles, a last tile of
    one row or of all, chunks, and one row more than 32."""
    w = chunked_workload(N + n_global, 1, N, 2, n_global)
    got, _ = hp.run_hip(w, True)
    print(hp.report(hp.compare(got, hp.run_oracle(w, True, [(0, 0), (0, 1)]), w, w.name)), flush=True)


@pytest.mark.parametrize("n_global,B,N,H", [(1, 72, 130, 2), (32, 70, 160, 2), (33, 70, 200, 2), (16, 65, 128, 2), (7, 50, 300, 2),
                                            (32, 54, 300, 2), (8, 42, 500, 2), (60, 42, 500, 2)])
def test_forward_of_launches_that_fill_half_of_the_chip(n_global, B, N, H):
    """Such owners where a launch has one, two, three or four tiles of owners a sequence and about two units a compute unit,
    in either order of its units."""
    w = chunked_workload(N + n_global, B, N, H, n_global)
    got, _ = hp.run_hip(w, False)
    pairs = [(b, h) for b in (0, B // 2, B - 1) for h in range(H)]
    print(hp.report(hp.compare(got, hp.run_oracle(w, False, pairs), w, w.name)), flush=True)
