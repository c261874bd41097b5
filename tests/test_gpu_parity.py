"""GPU parity: the HIP path, called through the C ABI, against the CPU oracle.

Bars: attention slice within 1e-5 (fp32 storage) / 2e-2 (bf16 storage, fp32
accumulate) of the oracle's unrounded float64 result, normwise and elementwise
(see gpu_util.assert_att_close); identity channels bit-exact; DK within 1e-5.
"""
import numpy as np
import pytest
import torch

from paper_2503_06671_amd import binding, workloads as wk
from tests import gpu_util as gu

pytestmark = pytest.mark.gpu

F32, BF16 = wk.F32, wk.BF16


def check_forward(wl, oracle, what=None):
    what = what or wl.name
    print(f"[case] {what}", flush=True)
    ref_att, ref_dk, _ = oracle.forward_workload(wl, want_out=False)
    out = gu.run_forward(wl)
    gu.assert_identity_bits(out, wl, what)
    rel = gu.assert_att_close(gu.att_as_f64(out, wl), ref_att, wl.dtype, what)
    dk = gu.run_dk(wl)
    gu.assert_dk_close(dk, ref_dk, what)
    return rel


# ------------------------------------------------------------------ small shapes, every Ks

@pytest.mark.parametrize("Ks", list(range(1, 32, 2)))
def test_every_kernel_size_ragged_multi_tile(oracle, Ks):
    # 3 column tiles and 3 row tiles with ragged tails; x has a non-zero mean so DK is O(1)
    wl = wk.make_random(200 + Ks, 2, 6, 70, 150, 3, Ks, dtype=F32, x_mean=0.5)
    check_forward(wl, oracle)


@pytest.mark.parametrize("Ks", list(range(1, 32, 2)))
def test_bf16_storage_ragged_multi_tile(oracle, Ks):
    # every kernel size with bf16 storage: the matrix-core path up to Ks = 17 (its alignment
    # constants depend on Ks), the widened path beyond
    wl = wk.make_random(300 + Ks, 2, 5, 45, 136, 4, Ks, dtype=BF16, x_mean=0.5)
    check_forward(wl, oracle)


@pytest.mark.parametrize("N,C,H,W,Ca,Ks,dtype", [
    (1, 3, 2, 3, 3, 31, F32),      # image smaller than the kernel, Ca == C
    (2, 4, 5, 5, 2, 13, F32),      # odd plane size: unaligned planes, scalar stores and copy
    (2, 4, 5, 5, 2, 13, BF16),
    (1, 5, 1, 1, 2, 7, F32),       # a single pixel
    (3, 7, 9, 130, 5, 9, BF16),    # W % 4 == 2
    (1, 2, 33, 66, 1, 5, F32),     # W % 4 == 2, two column tiles
    (1, 4, 1, 257, 2, 3, BF16),    # one row, W odd
    (2, 3, 129, 3, 1, 17, F32),    # tall and thin
    (300, 2, 6, 6, 1, 3, F32),     # many small images
])
def test_edge_shapes(oracle, N, C, H, W, Ca, Ks, dtype):
    wl = wk.make_random(400 + H + W, N, C, H, W, Ca, Ks, dtype=dtype, x_mean=-0.25)
    check_forward(wl, oracle)


def test_plane_with_more_pool_tiles_than_one_polling_round(oracle):
    # 66 x 66 = 4356 pool tiles per plane: the gen item has to stage a channel's partial
    # sums in more than one round; a second channel and a ragged tail on both axes
    wl = wk.make_random(21, 1, 2, 2100, 4200 - 6, 2, 3, dtype=F32, x_mean=0.25)
    check_forward(wl, oracle)


def test_no_attention_channels_is_a_pure_copy(oracle):
    wl = wk.make_random(7, 2, 5, 17, 19, 0, 13)
    out = gu.run_forward(wl)
    assert np.array_equal(out.view(np.uint8), wl.x.view(np.uint8))


# Rows of whole runs of four elements, in bf16 half a 16-byte piece: planes that are whole pieces and planes that are not
# (odd heights), matrix and other kernel sizes, short and long calls, pool items and carried copies among them.
@pytest.mark.parametrize("dtype", [F32, BF16])
@pytest.mark.parametrize("N,H,W,Ks", [(2, 6, 4, 3), (2, 7, 4, 13), (1, 34, 12, 17), (1, 40, 60, 1), (3, 33, 68, 13), (1, 66, 76, 31),
                                      (1, 180, 324, 7), (1, 290, 324, 13), (40, 64, 60, 13), (61, 62, 60, 17), (1, 530, 260, 13)])
def test_rows_of_runs_of_four(oracle, dtype, N, H, W, Ks):
    wl = wk.make_random(380 + W + H, N, 19, H, W, 16, Ks, dtype=dtype, x_mean=0.3)
    check_forward(wl, oracle, f"{N}x{H}x{W} ks{Ks}")


# Copies of odd widths (no attention channels): less than one 16-byte access, one, less than one 16 KiB piece, several of
# them with a rest and a ragged end; and short calls beside conv items, whose copy items make one access at a time.
@pytest.mark.parametrize("dtype", [F32, BF16])
@pytest.mark.parametrize("N,C,Ca,H,W", [(1, 1, 0, 1, 3), (3, 1, 0, 1, 7), (2, 1, 0, 1, 9), (1, 3, 0, 33, 31), (2, 5, 0, 91, 61),
                                        (1, 16, 0, 1001, 1003), (1, 17, 1, 65, 63), (2, 21, 2, 47, 97), (1, 5, 4, 7, 3)])
def test_copies_of_odd_widths(oracle, dtype, N, C, Ca, H, W):
    wl = wk.make_random(370 + W, N, C, H, W, Ca, 5, dtype=dtype, x_mean=0.3)
    if Ca:
        check_forward(wl, oracle, f"{N}x{C}x{H}x{W} Ca={Ca}")
    else:
        assert np.array_equal(gu.run_forward(wl, use_gen=False).view(np.uint8), wl.x.view(np.uint8))


# Rows fetched, pooled and stored in pieces wherever they end: widths round the pieces' and the tiles' lengths, identity
# ranges of any number of bytes (carried by conv items, too: the last case fills every block slot with them).
@pytest.mark.parametrize("dtype", [F32, BF16])
@pytest.mark.parametrize("N,H,W,Ks", [(2, 5, 1, 3), (1, 7, 3, 7), (3, 7, 4, 13), (1, 5, 5, 1), (2, 33, 7, 13), (2, 33, 8, 13),
                                      (1, 9, 9, 31), (3, 37, 15, 13), (1, 67, 59, 17), (2, 33, 63, 13), (1, 40, 65, 7),
                                      (1, 33, 71, 31), (1, 70, 127, 13), (2, 31, 129, 17), (1, 257, 259, 13), (61, 63, 63, 13)])
def test_widths_round_the_pieces(oracle, dtype, N, H, W, Ks):
    wl = wk.make_random(350 + W, N, 19, H, W, 16, Ks, dtype=dtype, x_mean=0.3)
    check_forward(wl, oracle, f"{N}x{H}x{W} ks{Ks}")


@pytest.mark.parametrize("dtype", [F32, BF16])
@pytest.mark.parametrize("Ks", list(range(1, 18, 2)))
def test_tall_register_block_variant_ragged(oracle, Ks, dtype):
    # 6 x 16 planes of 3 x 2 tall tiles = 576 tiles >= two per compute unit: the library picks
    # the 4-row register block (64 x 64 tiles) by shape; ragged in H and W
    wl = wk.make_random(800 + Ks, 6, 17, 70, 150, 16, Ks, dtype=dtype, x_mean=0.5)
    check_forward(wl, oracle)


@pytest.mark.parametrize("dtype,Ks,N", [(F32, 13, 2), (BF16, 13, 2), (BF16, 31, 2), (F32, 5, 40), (BF16, 7, 40)])
def test_base_pointers_off_the_vector_alignment(oracle, dtype, Ks, N):
    # W % 4 == 0, but x and out start one element past a 16-byte boundary (views into larger
    # buffers): the tile loads, the row stores and the pass-through copy must all take their
    # element-wise forms.  N = 40 reaches the 4-row register block and the queue-dealt deal.
    wl = wk.make_random(820 + Ks, N, 7, 40, 72, 4, Ks, dtype=dtype, x_mean=0.4)
    print(f"[case] unaligned base, {wl.name}", flush=True)
    ref_att, _, _ = oracle.forward_workload(wl, want_out=False)
    x_al = gu.to_dev_x(wl.x, wl.dtype)
    numel = x_al.numel()
    for x_shift, out_shift in ((1, 1), (1, 0), (0, 3)):
        xb = torch.zeros(numel + 8, dtype=x_al.dtype, device="cuda")
        ob = torch.full((numel + 8,), float("nan"), dtype=x_al.dtype, device="cuda")
        x = xb[x_shift:x_shift + numel].view(x_al.shape)
        x.copy_(x_al)
        out = ob[out_shift:out_shift + numel].view(x_al.shape)
        assert x.data_ptr() % 16 == (x_shift * x.element_size()) % 16
        ws = binding.new_workspace(wl.N, wl.Ca, wl.H, wl.W)
        binding.convattn_forward(x, wl.Ca, gu.dev(wl.lk), ws, gen=gu.gen_params(wl), out=out)
        assert binding.workspace_errors(ws) == 0
        got = gu.out_to_np(out, wl.dtype)
        gu.assert_identity_bits(got, wl, "unaligned base")
        gu.assert_att_close(gu.att_as_f64(got, wl), ref_att, wl.dtype, "unaligned base")
        # nothing outside the view was written
        edge = ob.view(torch.int16 if dtype == BF16 else torch.int32)
        nan_bits = torch.full((1,), float("nan"), dtype=x_al.dtype).view(edge.dtype).item()
        assert all(int(v) == nan_bits for v in edge[:out_shift].tolist() + edge[out_shift + numel:].tolist())


@pytest.mark.parametrize("dtype,Ks", [(F32, 13), (BF16, 13), (F32, 3), (BF16, 31)])
def test_large_kernel_channel_stride_wider_than_the_kernel(oracle, dtype, Ks):
    # channel c's filter starts at lk + c * (Ks*Ks + 3): the gaps are filled with NaN and must
    # never be read into the result
    wl = wk.make_random(840 + Ks, 2, 6, 40, 72, 4, Ks, dtype=dtype, x_mean=0.3)
    ref_att, _, _ = oracle.forward_workload(wl, want_out=False)
    stride = Ks * Ks + 3
    flat = np.full((wl.Ca, stride), np.nan, np.float32)
    flat[:, :Ks * Ks] = wl.lk.reshape(wl.Ca, -1)
    x = gu.to_dev_x(wl.x, wl.dtype)
    out = torch.full_like(x, float("nan"))
    ws = binding.new_workspace(wl.N, wl.Ca, wl.H, wl.W)
    binding.convattn_forward(x, wl.Ca, gu.dev(flat), ws, gen=gu.gen_params(wl), out=out, ks=Ks,
                             lk_channel_stride=stride)
    assert binding.workspace_errors(ws) == 0
    got = gu.out_to_np(out, wl.dtype)
    gu.assert_identity_bits(got, wl, "wide channel stride")
    gu.assert_att_close(gu.att_as_f64(got, wl), ref_att, wl.dtype, "wide channel stride")


@pytest.mark.parametrize("Ca,hidden,bias,dtype", [(16, 8, False, F32), (16, 4, True, BF16), (48, 24, True, F32)])
def test_two_layer_estimator(oracle, Ca, hidden, bias, dtype):
    # the paper's estimator: 1x1 down, GELU, 1x1 up (hidden 8 / 4 / 24 in its variants)
    wl = wk.make_random(500 + hidden, 2, Ca + 4, 40, 72, Ca, 13, dtype=dtype, hidden=hidden, bias=bias,
                        x_mean=0.7)
    check_forward(wl, oracle)


@pytest.mark.parametrize("N,Ca,hidden,bias,dtype", [(40, 16, 8, True, F32), (12, 48, 24, True, BF16)])
def test_two_layer_estimator_run_by_the_conv_items(oracle, N, Ca, hidden, bias, dtype):
    # more conv items than resident blocks and few pool tiles per image: pool items, and the
    # conv items run the estimator themselves (weights staged in LDS for the small
    # estimator, read from memory for the wide one)
    wl = wk.make_random(520 + hidden, N, Ca + 4, 40, 72, Ca, 5, dtype=dtype, hidden=hidden, bias=bias,
                        x_mean=0.7)
    check_forward(wl, oracle)


@pytest.mark.parametrize("dtype", [F32, BF16])
def test_two_layer_estimator_large_planes(oracle, dtype):
    # 11 x 7 pool tiles x 8 channels > 512 mailboxes per image: channel-mean items, and the
    # conv items run the two-layer estimator from the collected means
    wl = wk.make_random(530, 2, 10, 200, 704, 8, 13, dtype=dtype, hidden=4, bias=True, x_mean=0.4)
    check_forward(wl, oracle)


def test_many_small_images_beyond_one_round(oracle):
    # 3200 conv items of short tap loops: pool items, queue-dealt blocks, and conv items that
    # collect the pool sums themselves
    wl = wk.make_random(540, 200, 8, 40, 40, 8, 3, dtype=F32, x_mean=0.3)
    check_forward(wl, oracle)


@pytest.mark.parametrize("C", [40, 10])
def test_queue_dealt_call_with_lopsided_conv_and_copy_shares(oracle, C):
    # 1280 conv items (more than fit at once) beside many copy items (C = 40) or few (C = 10):
    # the layers in which the two kinds alternate follow their counts
    wl = wk.make_random(541, 160, C, 40, 40, 8, 5, dtype=F32, x_mean=0.2)
    check_forward(wl, oracle)


def test_shared_single_filter(oracle):
    wl = wk.make_random(11, 2, 6, 30, 70, 4, 13)
    one = wl.lk[2].copy()
    print("[case] shared filter", flush=True)
    x = gu.to_dev_x(wl.x, wl.dtype)
    out = torch.empty_like(x)
    binding.convattn_forward(x, 4, gu.dev(one), binding.new_workspace(2, 4, 30, 70), out=out)
    torch.cuda.synchronize()
    ref, _, _ = oracle.convattn_forward(wl.x, 4, one, want_out=False)
    gu.assert_att_close(gu.att_as_f64(out.cpu().numpy(), wl), ref, F32, "shared filter")


# ------------------------------------------------------------------ exact special cases on the GPU

@pytest.mark.parametrize("dtype", [F32, BF16])
def test_delta_kernel_is_exact_identity(dtype):
    wl = wk.make_random(12, 2, 5, 50, 90, 3, 13, dtype=dtype)
    lk = np.zeros((3, 13, 13), np.float32)
    lk[:, 6, 6] = 1.0
    out = gu.run_forward(wl, use_gen=False, lk=lk)
    assert np.array_equal(out.view(np.uint8), wl.x.view(np.uint8))
    # and through the dynamic path: LK = 0, DK = centre delta
    dk = np.zeros((2, 3, 3, 3), np.float32)
    dk[:, :, 1, 1] = 1.0
    out = gu.run_forward(wl, use_gen=False, lk=np.zeros_like(lk), dk_in=dk)
    assert np.array_equal(out.view(np.uint8), wl.x.view(np.uint8))


@pytest.mark.parametrize("dtype,Ks", [(F32, 13), (BF16, 13), (F32, 31), (F32, 5)])
def test_ones_conv_ones_is_exact(dtype, Ks):
    H, W, p = 40, 100, (Ks - 1) // 2
    wl = wk.make_random(13, 1, 2, H, W, 1, Ks, dtype=dtype)
    ones = np.ones((1, 2, H, W), np.float32)
    wl.x = wk.f32_to_bf16_bits(ones) if dtype == BF16 else ones
    out = gu.run_forward(wl, use_gen=False, lk=np.ones((1, Ks, Ks), np.float32))
    cnt = lambda L, t: min(t, p) + min(L - 1 - t, p) + 1
    want = np.array([[cnt(H, y) * cnt(W, x) for x in range(W)] for y in range(H)], float)
    assert np.array_equal(gu.att_as_f64(out, wl)[0, 0], want)


def test_off_centre_delta_shift():
    wl = wk.make_random(14, 1, 2, 40, 100, 1, 7)
    lk = np.zeros((1, 7, 7), np.float32)
    lk[0, 1, 5] = 1.0            # out[y,x] = x[y-2, x+2]
    out = gu.run_forward(wl, use_gen=False, lk=lk)
    want = np.zeros((40, 100), np.float32)
    want[2:, :-2] = wl.x[0, 0, :-2, 2:]
    assert np.array_equal(out[0, 0], want)


def test_generated_dk_equals_given_dk_bit_for_bit():
    wl = wk.make_random(15, 3, 6, 50, 70, 4, 13, x_mean=0.5)
    full = gu.run_forward(wl)
    dk = gu.run_dk(wl)
    two_step = gu.run_forward(wl, use_gen=False, dk_in=dk)
    assert np.array_equal(full.view(np.uint8), two_step.view(np.uint8))


def test_batch_equals_single_images_bit_for_bit():
    wl = wk.make_random(16, 3, 5, 37, 80, 3, 13, dtype=BF16, x_mean=0.3)
    full = gu.run_forward(wl)
    dk = gu.run_dk(wl)
    for n in range(3):
        one = wk.make_random(16, 3, 5, 37, 80, 3, 13, dtype=BF16, x_mean=0.3)
        one.x = np.ascontiguousarray(wl.x[n:n + 1]); one.N = 1
        assert np.array_equal(gu.run_forward(one)[0], full[n])
        assert np.array_equal(gu.run_dk(one)[0], dk[n])


def test_one_workspace_serves_a_sequence_of_different_calls():
    # One workspace, sized for the largest shape, through calls that take every estimator
    # form, both dealing schemes and both entry points, twice over: each result must equal,
    # bit for bit, what the same call gives in a workspace of its own.
    cases = [
        wk.make_random(601, 2, 6, 40, 72, 4, 5, dtype=F32, x_mean=0.4),                 # conv items run the estimator
        wk.make_random(602, 2, 6, 40, 72, 4, 13, dtype=BF16, x_mean=0.4),               # gen items, DK picked up in the loop
        wk.make_random(603, 1, 10, 200, 704, 8, 13, dtype=F32, hidden=4, x_mean=0.4),   # channel means, one round
        wk.make_random(604, 3, 12, 150, 400, 8, 7, dtype=BF16, x_mean=0.4),             # pool items, queue-dealt blocks
        wk.make_random(605, 2, 5, 17, 19, 0, 13, dtype=F32),                            # copy only
        wk.make_random(606, 40, 6, 30, 30, 4, 3, dtype=F32, x_mean=0.4),                # many small images
    ]
    size = max(binding.workspace_bytes(w.N, w.Ca, w.H, w.W) for w in cases)
    ws = torch.empty(size, dtype=torch.uint8, device="cuda")
    binding.workspace_init(ws)
    alone = [(gu.run_forward(w), gu.run_dk(w) if w.Ca > 0 else None) for w in cases]
    for rnd in range(2):
        for w, (out_alone, dk_alone) in zip(cases, alone):
            print(f"[case] shared workspace, round {rnd}, {w.name}", flush=True)
            assert np.array_equal(gu.run_forward(w, ws=ws).view(np.uint8), out_alone.view(np.uint8))
            if w.Ca > 0:
                assert np.array_equal(gu.run_dk(w, ws=ws), dk_alone)
                two_step = gu.run_forward(w, use_gen=False, dk_in=dk_alone, ws=ws)
                assert np.array_equal(two_step.view(np.uint8), out_alone.view(np.uint8))


@pytest.mark.parametrize("N,C,H,W,Ca,Ks", [
    (2, 6, 70, 132, 4, 3), (2, 6, 70, 132, 4, 9), (2, 6, 70, 132, 4, 13), (2, 6, 70, 132, 4, 17),   # two-row blocks
    (8, 10, 130, 132, 8, 13), (8, 10, 130, 140, 8, 7),                                              # four-row blocks
])
def test_bf16_matrix_path_eight_byte_tile_fetch(oracle, N, C, H, W, Ca, Ks):
    # W % 4 == 0 but W % 8 != 0: the matrix-core path fetches its tile in 4-element chunks
    # (16-byte pieces need W % 8 == 0, single elements serve every other width)
    wl = wk.make_random(900 + Ks + W, N, C, H, W, Ca, Ks, dtype=BF16, x_mean=0.4)
    check_forward(wl, oracle)


@pytest.mark.parametrize("dtype", [F32, BF16])
@pytest.mark.parametrize("hidden,bias", [(0, True), (8, True), (16, False)])
def test_large_planes_in_one_round_conv_items_run_the_estimator_from_the_channel_means(oracle, dtype, hidden, bias):
    # more pool mailboxes per image than one item collects (8 channels x 77 tiles), a small
    # estimator, and all conv items resident at once: gsum items publish the channel means and
    # every conv item runs its nine estimator outputs itself
    wl = wk.make_random(920 + hidden, 1, 10, 200, 704, 8, 13, dtype=dtype, hidden=hidden, bias=bias, x_mean=0.4)
    check_forward(wl, oracle)


def test_captured_graph_replays_like_plain_calls():
    # Three different calls on one workspace captured into one graph; the graph is replayed
    # several times with plain calls and synchronisations in between, and every replay must
    # reproduce the plain calls' outputs bit for bit (the call tag lives on the device, so a
    # replay is a new call).
    cases = [
        wk.make_random(611, 2, 6, 40, 72, 4, 13, dtype=F32, x_mean=0.4),
        wk.make_random(612, 1, 10, 200, 704, 8, 13, dtype=BF16, x_mean=0.4),
        wk.make_random(613, 3, 12, 150, 400, 8, 7, dtype=F32, x_mean=0.4),
    ]
    size = max(binding.workspace_bytes(w.N, w.Ca, w.H, w.W) for w in cases)
    ws = torch.empty(size, dtype=torch.uint8, device="cuda")
    binding.workspace_init(ws)
    xs = [gu.to_dev_x(w.x, w.dtype) for w in cases]
    lks = [gu.dev(w.lk) for w in cases]
    gens = [gu.gen_params(w) for w in cases]
    want = [gu.run_forward(w) for w in cases]
    outs = [torch.empty_like(x) for x in xs]
    stream = torch.cuda.Stream()

    def enqueue():
        for w, x, lk, gen, out in zip(cases, xs, lks, gens, outs):
            binding.convattn_forward(x, w.Ca, lk, ws, gen=gen, out=out, stream=stream)

    with torch.cuda.stream(stream):
        enqueue()
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=stream):
        enqueue()
    for rep in range(4):
        for out in outs:
            out.fill_(float("nan"))
        torch.cuda.synchronize()
        with torch.cuda.stream(stream):
            graph.replay()
        torch.cuda.synchronize()
        assert binding.workspace_errors(ws, stream) == 0
        for w, out, ref in zip(cases, outs, want):
            print(f"[case] graph replay {rep}, {w.name}", flush=True)
            assert np.array_equal(gu.out_to_np(out, w.dtype).view(np.uint8), ref.view(np.uint8))
        # plain work on the same workspace between replays
        with torch.cuda.stream(stream):
            binding.convattn_forward(xs[rep % 3], cases[rep % 3].Ca, lks[rep % 3], ws, gen=gens[rep % 3],
                                     out=outs[rep % 3], stream=stream)
        torch.cuda.synchronize()


@pytest.mark.parametrize("dtype", [F32, BF16])
def test_planted_non_finite_values_in_identity_channels(oracle, dtype):
    wl = wk.make_random(17, 2, 6, 20, 36, 2, 7, dtype=dtype)
    flat = wl.x.reshape(2, 6, -1)
    if dtype == F32:
        u = flat.view(np.uint32)
        u[0, 3, 0], u[0, 4, 1], u[1, 5, 2], u[1, 2, 3] = 0x7FC00001, 0xFF800000, 0x00000001, 0x7FA00000
    else:
        flat[0, 3, 0], flat[0, 4, 1], flat[1, 5, 2], flat[1, 2, 3] = 0x7FC1, 0xFF80, 0x0001, 0x7FA0
    check_forward(wl, oracle, "planted non-finite")


@pytest.mark.parametrize("dtype,Ks", [(F32, 13), (F32, 31), (BF16, 21), (BF16, 13), (BF16, 5), (BF16, 17)])
def test_non_finite_pixels_in_the_attention_slice(oracle, dtype, Ks):
    # Where do NaN/Inf pixels of the attention slice show in the output?  The definition
    # (and the oracle): at every output whose Ks x Ks window (or DK's 3 x 3) covers the pixel.
    # fp32 storage, and bf16 storage with Ks >= 19, must give exactly that footprint.  The
    # matrix path (bf16 storage, Ks <= 17) forms 16 neighbouring outputs of a row from the 32
    # tile columns that start P + A columns left of the first (A pads the halo to 8 columns),
    # most of them times a zero of the band: there the footprint may widen, inside the rows
    # the definition reaches, to every 16-column block whose 32 columns hold the pixel - and
    # no further.  Everything else stays within the usual bar.
    wl = wk.make_random(860 + Ks, 2, 5, 50, 150, 3, Ks, dtype=dtype)
    rng = np.random.default_rng(861)
    dk = rng.standard_normal((2, 3, 3, 3)).astype(np.float32)
    spots = [(0, 0, 0, 0, "inf"), (0, 1, 25, 70, "nan"), (1, 2, 49, 149, "-inf"), (1, 0, 13, 64, "nan"),
             (0, 2, 31, 127, "inf")]
    xf = wl.x_as_f32().copy()
    for n, c, y, x_, kind in spots:
        xf[n, c, y, x_] = {"inf": np.inf, "-inf": -np.inf, "nan": np.nan}[kind]
    wl.x = wk.f32_to_bf16_bits(xf) if dtype == BF16 else xf
    with np.errstate(invalid="ignore"):
        ref_att, _, _ = oracle.convattn_forward(wl.x, wl.Ca, wl.lk, wl.dtype, dk_in=dk, want_out=False)
    out = gu.run_forward(wl, use_gen=False, dk_in=dk)
    gu.assert_identity_bits(out, wl, "non-finite attention pixels")
    got = gu.att_as_f64(out, wl)
    bad_ref, bad_got = ~np.isfinite(ref_att), ~np.isfinite(got)
    p = (Ks - 1) // 2
    assert bad_ref.sum() >= len(spots) * (p + 1) ** 2
    matrix = dtype == BF16 and Ks <= 17
    if matrix:
        ph = max(p, 1)
        pad = ph + (8 - ph % 8) % 8
        wider = bad_ref.copy()
        for n, c, y, x_, _ in spots:
            for X0 in range(0, wl.W, 16):
                if X0 - pad <= x_ <= X0 - pad + 31:
                    wider[n, c, max(0, y - p):y + p + 1, X0:X0 + 16] = True
        assert not (bad_ref & ~bad_got).any(), "a non-finite result of the definition came out finite"
        assert not (bad_got & ~wider).any(), "NaN outside the blocks whose input columns hold the pixel"
    else:
        assert np.array_equal(bad_ref, bad_got), "NaN/Inf footprint differs from the definition's"
    ok = ~bad_got
    tol = gu.TOL[dtype]
    fin = ref_att[~bad_ref]
    scale, rms = np.abs(fin).max(), float(np.sqrt(np.mean(fin ** 2)))
    d = np.abs(got[ok] - ref_att[ok])
    assert d.max() <= tol * scale
    assert (d <= tol * (np.abs(ref_att[ok]) + rms)).all()


@pytest.mark.parametrize("dtype,Ks,N,H,W", [(F32, 15, 1, 33, 66), (F32, 17, 1, 65, 129), (F32, 17, 24, 64, 65), (F32, 19, 1, 31, 64),
                                            (F32, 31, 2, 40, 80), (BF16, 19, 1, 32, 72), (BF16, 31, 1, 33, 64)])
def test_large_kernels_at_any_scale(oracle, dtype, Ks, N, H, W):
    # values and weights of every size, a plane of zeros, planes whose sizes lie 2^40 apart, weights too large for
    # the terms and a NaN (both: the vector loop).  fp32 storage, in the 2-norm: fp32 products and sums stay within sqrt(2 taps) 2^-24 of
    # terms whose squares add up to the result's, and two terms are within 2^-23 of each factor.
    base = wk.make_random(920 + Ks, N, 6, H, W, 4, Ks, dtype=dtype)
    dk0 = np.random.default_rng(921).standard_normal((N, 4, 3, 3)).astype(np.float32)
    planes = np.array([1.0, 0.0, 2.0 ** 20, 2.0 ** -20]).reshape(1, 4, 1, 1)
    for what, fx, fw in (("ordinary", 1.0, 1.0), ("small", 2.0 ** -90, 2.0 ** -20), ("large", 2.0 ** 90, 2.0 ** -30),
                         ("small x large", 2.0 ** -100, 2.0 ** 100), ("beyond", 2.0 ** -60, 2.0 ** 110), ("planes", planes, 1.0), ("nan", 1.0, 1.0)):
        print(f"[case] {what} {dtype} Ks={Ks}", flush=True)
        xf = base.x_as_f32().copy()
        xf[:, :4] = (xf[:, :4] * fx).astype(np.float32)
        if what == "nan":
            xf[0, 1, H // 2, W // 2] = np.nan
        x = wk.f32_to_bf16_bits(xf) if dtype == BF16 else xf
        wl = wk.make_random(920 + Ks, N, 6, H, W, 4, Ks, dtype=dtype)
        wl.x, wl.lk = x, (base.lk * fw).astype(np.float32)
        dk = (dk0 * fw).astype(np.float32)
        ref, _, _ = oracle.convattn_forward(x, 4, wl.lk, dtype, dk_in=dk, want_out=False)
        got = gu.att_as_f64(gu.run_forward(wl, use_gen=False, dk_in=dk), wl)
        assert np.array_equal(np.isnan(ref), np.isnan(got)), what
        for c in range(4):
            r, g = ref[:, c], got[:, c]
            ok = ~np.isnan(r)
            rms = np.sqrt((r[ok] ** 2).mean())
            err = np.sqrt(((g - r)[ok] ** 2).mean())
            bound = (np.sqrt(2 * Ks * Ks) + 4) * 2.0 ** -24 if dtype == F32 else 2.0 ** -8
            assert err <= bound * rms, (what, c, err / rms, bound)


@pytest.mark.parametrize("dtype,Ks,N,H,W", [(F32, 15, 1, 33, 66), (F32, 17, 1, 65, 129), (F32, 17, 24, 64, 65), (F32, 19, 1, 31, 64),
                                            (F32, 31, 2, 40, 80), (BF16, 19, 1, 32, 72), (BF16, 31, 1, 33, 64)])
def test_large_kernels_of_wide_range(oracle, dtype, Ks, N, H, W):
    # magnitudes far apart inside a tile or a kernel.  Every output lies within its own terms' bound - Ks^2 + 9 products and
    # additions, each within 2^-23 of the magnitudes summed, and eight more for the terms of both factors - and those
    # whose window does not reach the large values are as near as without them.
    base = wk.make_random(925 + Ks, N, 4, H, W, 4, Ks, dtype=dtype)
    dk = np.random.default_rng(926).standard_normal((N, 4, 3, 3)).astype(np.float32)
    rng = np.random.default_rng(927)
    centre = np.zeros((Ks, Ks))
    centre[Ks // 2, Ks // 2] = 1.0
    sparse = np.where(rng.random(base.x.shape) < 0.01, 1.0, 0.0)
    for what, large, fx, fw in (("1e8", 1e8, 1.0, 1.0), ("1e12", 1e12, 1.0, 1.0), ("1e30", 1e30, 1.0, 1.0), ("2^27 apart", 2.0 ** 27, 1.0, 1.0),
                                ("any size", 1.0, 2.0 ** rng.integers(-60, 60, base.x.shape), 1.0),
                                ("weights 2^-45", 1.0, sparse, centre + 2.0 ** -45 * (1 - centre)),
                                ("weights 2^-30", 1.0, sparse, centre + 2.0 ** -30 * (1 - centre))):
        print(f"[case] {what} {dtype} Ks={Ks}", flush=True)
        xf = (base.x_as_f32() * fx).astype(np.float32)
        if large != 1.0:
            xf[0, 1, 2, 3] = large
            xf[N - 1, 2, H - 1, W - 1] = -large
        wl = wk.make_random(925 + Ks, N, 4, H, W, 4, Ks, dtype=dtype)
        wl.x, wl.lk = (wk.f32_to_bf16_bits(xf) if dtype == BF16 else xf), (base.lk * fw).astype(np.float32)
        d = (dk * (2.0 ** -45 if "weights" in what else 1.0)).astype(np.float32)
        ref, _, _ = oracle.convattn_forward(wl.x, 4, wl.lk, dtype, dk_in=d, want_out=False)
        ax = wl.x & 0x7fff if dtype == BF16 else np.abs(wl.x)
        mags, _, _ = oracle.convattn_forward(ax, 4, np.abs(wl.lk), dtype, dk_in=np.abs(d), want_out=False)
        got = gu.att_as_f64(gu.run_forward(wl, use_gen=False, dk_in=d), wl)
        bound = (Ks * Ks + 17) * 2.0 ** -23 * mags + (2.0 ** -8 * np.abs(ref) if dtype == BF16 else 0.0)
        assert (np.abs(got - ref) <= bound).all(), (what, (np.abs(got - ref) / bound).max())
    # a kernel of a single one moves the values as they are
    xf = np.sign(base.x_as_f32()) * (1.0 + rng.random(base.x.shape))
    mixed = (xf * 2.0 ** rng.integers(-13, 15, xf.shape)).astype(np.float32)
    wl.x = wk.f32_to_bf16_bits(mixed) if dtype == BF16 else mixed
    wl.lk = np.array(np.broadcast_to(centre, base.lk.shape), np.float32)
    assert np.array_equal(gu.run_forward(wl, use_gen=False)[:, :4], wl.x[:, :4])
    # five by four taps; values of 2^-13 in the left half and of 2^14 in the right: the widest range the terms are used for
    xf = (xf * np.where(np.arange(W) < W // 2, 2.0 ** -13, 2.0 ** 14)).astype(np.float32)
    wl.x = wk.f32_to_bf16_bits(xf) if dtype == BF16 else xf
    wl.lk[:, Ks // 2 - 2:Ks // 2 + 3, Ks // 2 - 2:Ks // 2 + 2] = rng.standard_normal((4, 5, 4))
    ref, _, _ = oracle.convattn_forward(wl.x, 4, wl.lk, dtype, want_out=False)
    mags, _, _ = oracle.convattn_forward(wl.x & 0x7fff if dtype == BF16 else np.abs(wl.x), 4, np.abs(wl.lk), dtype, want_out=False)
    got = gu.att_as_f64(gu.run_forward(wl, use_gen=False), wl)
    assert (np.abs(got - ref) <= (20 + 8) * 2.0 ** -23 * mags + (2.0 ** -8 * np.abs(ref) if dtype == BF16 else 0.0)).all()


@pytest.mark.parametrize("dtype,Ks", [(F32, 15), (F32, 17), (F32, 31), (BF16, 19), (BF16, 31)])
def test_large_kernels_with_dk_of_any_size(oracle, dtype, Ks):
    # DK of up to 2^120 and weights of up to 2^125 on values whose products are ordinary numbers
    wl = wk.make_random(935 + Ks, 1, 4, 33, 70, 4, Ks, dtype=dtype)
    dk = np.random.default_rng(936).standard_normal((1, 4, 3, 3)).astype(np.float32)
    x0, lk0 = wl.x_as_f32(), wl.lk.copy()
    for what, fx, fw, fd in (("dk", 2.0 ** -100, 1.0, 2.0 ** 120), ("weights", 2.0 ** -100, 2.0 ** 125, 2.0 ** 100), ("large x", 2.0 ** 100, 2.0 ** -120, 2.0 ** -110)):
        print(f"[case] {what} {dtype} Ks={Ks}", flush=True)
        xf = (x0 * fx).astype(np.float32)
        wl.x, wl.lk, d = (wk.f32_to_bf16_bits(xf) if dtype == BF16 else xf), (lk0 * fw).astype(np.float32), (dk * fd).astype(np.float32)
        ref, _, _ = oracle.convattn_forward(wl.x, 4, wl.lk, dtype, dk_in=d, want_out=False)
        gu.assert_att_close(gu.att_as_f64(gu.run_forward(wl, use_gen=False, dk_in=d), wl), ref, dtype, what)


def test_bf16_large_kernel_weight_rounding_error_bound(oracle):
    # With bf16 storage and Ks <= 17 the fp32 large-kernel weights are rounded to bf16 on
    # the device (operands of the bf16 matrix instructions).  Bound asserted here: the normwise error
    # against the float64 oracle stays below 6e-3 at Ks = 13 (the store's own rounding to
    # bf16 alone is 2^-9 ~ 2e-3 relative per value; weights add an independent 2^-9 per tap),
    # far inside the 2e-2 bar; with weights that are exactly representable in bf16 the
    # error is that of the store rounding alone.
    wl = wk.make_random(880, 2, 5, 96, 160, 4, 13, dtype=BF16, x_mean=0.0)
    rel = check_forward(wl, oracle, "bf16, fp32 weights")
    wl.lk = wk.bf16_bits_to_f32(wk.f32_to_bf16_bits(wl.lk))
    rel_exact = check_forward(wl, oracle, "bf16, bf16-exact weights")
    print(f"[bound] normwise error: fp32 weights {rel:.3e}, bf16-exact weights {rel_exact:.3e}", flush=True)
    assert rel <= 6e-3 and rel_exact <= 4.5e-3


def test_linearity_with_dk_fixed():
    wl = wk.make_random(18, 1, 3, 40, 70, 2, 13)
    rng = np.random.default_rng(19)
    x2 = rng.standard_normal(wl.x.shape).astype(np.float32)
    dk = rng.standard_normal((1, 2, 3, 3)).astype(np.float32)
    f = lambda x: (setattr(wl, "x", x), gu.run_forward(wl, use_gen=False, dk_in=dk))[1][:, :2].astype(np.float64)
    x1 = wl.x.copy()
    lhs = f((2.0 * x1 - 0.5 * x2).astype(np.float32))
    rhs = 2.0 * f(x1) - 0.5 * f(x2)
    assert np.abs(lhs - rhs).max() <= 2e-5 * np.abs(rhs).max()


# ------------------------------------------------------------------ the five benchmark workloads

def visible_dk_variants(wl):
    """Same workload with LK = 0, and with x shifted by 0.5 so DK is O(1)."""
    a = wk.make_config(int(wl.name[3]), wl.Ks if wl.name.startswith("cfg4") else None)
    a.lk = np.zeros_like(a.lk); a.name += "_lk0"
    b = wk.make_config(int(wl.name[3]), wl.Ks if wl.name.startswith("cfg4") else None)
    xf = b.x_as_f32() + np.float32(0.5)
    b.x = wk.f32_to_bf16_bits(xf) if b.dtype == BF16 else xf
    b.name += "_shift"
    return a, b


@pytest.mark.parametrize("idx", [0, 1, 2, 3])
def test_benchmark_workloads_full_size(oracle, idx):
    wl = wk.make_config(idx)
    check_forward(wl, oracle)
    for v in visible_dk_variants(wl):
        check_forward(v, oracle)


@pytest.mark.parametrize("Ks", wk.CFG4_KS)
def test_benchmark_workload_4_full_size(oracle, Ks):
    wl = wk.make_config(4, Ks)
    check_forward(wl, oracle)
    if Ks == 13:
        for v in visible_dk_variants(wl):
            check_forward(v, oracle)


def test_large_model_workload_full_size(oracle):
    # C = 192, 48 attention channels, estimator with a hidden layer of 24: 1440 conv items
    # (queue-dealt), channel-mean items, the two-layer estimator run by every conv item
    check_forward(wk.make_large_model(), oracle)


@pytest.mark.parametrize("N,C,H,W,Ca,hidden", [
    (1, 100, 20, 20, 100, 0),     # one wide linear layer: 900 output rows staged 64 at a time
    (1, 104, 96, 128, 100, 0),    # the same behind channel-mean items (600 pool mailboxes per image)
    (2, 60, 96, 128, 56, 32),     # two layers, channel means, two rounds of output rows
    (1, 200, 16, 16, 200, 200),   # too large to stage: weights read from memory
    (1, 200, 96, 128, 200, 64),   # the same behind channel-mean items, more means than polling threads
])
def test_estimators_beyond_the_small_ones(oracle, N, C, H, W, Ca, hidden):
    wl = wk.make_random(560 + Ca + hidden, N, C, H, W, Ca, 3, dtype=F32, hidden=hidden, bias=True, x_mean=0.5)
    check_forward(wl, oracle)

