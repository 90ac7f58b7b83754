"""GPU parity: the encoder workloads through the C ABI against the CPU oracle."""
from dataclasses import replace

import numpy as np
import pytest

import oracle as O
import vf_inputs as I
from vfharness import (TOL, check_against_oracle, check_independent_bound, check_update_from_own_gradient,
                       oracle_steps, run_gpu, weights_only_gradient)

pytestmark = pytest.mark.gpu

FUSED = 1
NO_GRAPH = 2


def _case(name, jitter=0.1):
    wl = I.workload(name)
    theta = I.make_params(wl, jitter=jitter)
    x, y = I.make_batch(wl)
    return wl, theta, x, y


@pytest.mark.parametrize("flags", [NO_GRAPH, 0, FUSED])
@pytest.mark.parametrize("name", ["enc_tiny_f32", "enc_small_f32", "enc_small_bf16", "enc_mid_bf16", "enc_vocab_f32",
                                  "enc_vocab_bf16", "enc_odd_f32", "enc_wide_bf16"])
def test_encoder_step_matches_oracle(name, flags):
    print(f"case {name} flags={flags}", flush=True)
    wl, theta, x, y = _case(name)
    gpu = run_gpu(wl, theta, x, y, flags=flags)
    ref = oracle_steps(wl, theta, x, y)
    # Adam: new parameters are compared through the device's own gradient (an entry whose
    # gradient is within rounding of zero moves by +lr on one side and -lr on the other)
    check_against_oracle(wl, gpu, ref)
    check_update_from_own_gradient(wl, gpu, theta, tol=1e-4)


@pytest.mark.parametrize("T", [1, 17, 33, 95, 100, 128, 130])
def test_encoder_sequence_lengths(T):
    """Sequences that do not fill the attention kernel's tiles of 32 tokens (130: the generic kernels)."""
    print(f"T={T}", flush=True)
    wl = replace(I.workload("enc_small_bf16"), name=f"enc_T{T}", seq_len=T, n_masked=max(1, int(0.15 * T)))
    theta = I.make_params(wl, jitter=0.1)
    x, y = I.make_batch(wl)
    ref = oracle_steps(wl, theta, x, y)
    base = run_gpu(wl, theta, x, y, flags=FUSED | NO_GRAPH)
    check_against_oracle(wl, base, ref)
    two = run_gpu(wl, theta, x, y, flags=FUSED | OVERLAP | NO_GRAPH)
    assert base["G"].tobytes() == two["G"].tobytes()


@pytest.mark.parametrize("T", [1, 17, 33, 100])
def test_workspace_of_sequences_that_fill_no_tile(T):
    """Stored probabilities take T rows of T rounded up to 8 per head, not whole tiles of 32 x 32.  The rest of the
    workspace grows with the tokens: a line through 32 and 64, where the tiles are full."""
    import paper_2009_09523_amd as vf
    from paper_2009_09523_amd.binding import config_from_workload
    layers, heads, sequences = 3, 2, 512

    def workspace(t, p):
        wl = replace(I.workload("enc_small_bf16"), name=f"enc_ws_T{t}", n_layers=layers, d_model=128, n_heads=heads, d_ffn=128,
                     seq_len=t, n_masked=1, node_sizes=(sequences,))
        eng = vf.VirtualNodeStep(config_from_workload(wl, flags=FUSED | NO_GRAPH))
        size = eng.workspace_bytes - layers * sequences * heads * 2 * t * p
        eng.close()
        return size
    a, b = workspace(32, 32), workspace(64, 64)
    pitch = (T + 7) // 8 * 8
    assert workspace(T, pitch) <= a + (T - 32) * (b - a) / 32 + (2 << 20)


@pytest.mark.parametrize("name,T,sizes", [("enc_small_f32", 5, (3, 1)), ("enc_small_f32", 70, (2, 1)),
                                          ("enc_small_f32", 130, (24,)), ("enc_small_bf16", 131, (22, 2))])
def test_generic_attention_products(name, T, sizes):
    """The batched products on the fp32 matrix instruction: contractions and tiles that are not filled, rows that
    allow no vector reads, one 16 x 16 tile per wavefront and (1024 and more of them) 32 x 32."""
    print(f"case {name} T={T} sizes={sizes}", flush=True)
    wl = replace(I.workload(name), name=f"{name}_T{T}", seq_len=T, n_masked=max(1, int(0.15 * T)), node_sizes=sizes)
    theta = I.make_params(wl, jitter=0.1)
    x, y = I.make_batch(wl)
    check_against_oracle(wl, run_gpu(wl, theta, x, y, flags=FUSED | NO_GRAPH), oracle_steps(wl, theta, x, y))


@pytest.mark.parametrize("sizes", [(4099, 4100, 4101, 4098), (3, 4100, 4101, 4098, 4100, 2)])
def test_units_of_more_heads_than_a_grid_has_rows(sizes):
    """Four nodes of different sizes go as one unit, whose attention products are then more than 65535 (16398
    sequences of four heads): each node alone has few enough."""
    print(f"sizes={sizes}", flush=True)
    wl = replace(I.workload("enc_small_f32"), name="enc_many", n_layers=1, d_model=16, n_heads=4, d_ffn=32, seq_len=2,
                 vocab=53, n_masked=1, node_sizes=sizes)
    theta = I.make_params(wl, jitter=0.1)
    x, y = I.make_batch(wl)
    gpu = run_gpu(wl, theta, x, y, flags=FUSED | NO_GRAPH, node_group=4)
    check_against_oracle(wl, gpu, oracle_steps(wl, theta, x, y))


@pytest.mark.parametrize("d", [8, 260, 512, 772, 1024])
@pytest.mark.parametrize("shared", [63, 64, 65, 257, 300])
def test_token_rows_that_many_tokens_share(d, shared):
    """The rows of an id with 64 tokens or more are added up by several workgroups, 256 columns each, 256 tokens at
    a time.  `shared` tokens of the first node carry one id, scattered, the second node's carry it once, and every
    other id has few.  One layer, so the table's gradient is the embedding's and the decoder's (tol: the harness')."""
    print(f"d={d} shared={shared}", flush=True)
    wl = replace(I.workload("enc_small_f32"), name=f"enc_shared_{d}_{shared}", n_layers=1, d_model=d, n_heads=2, d_ffn=16,
                 seq_len=19, vocab=211, n_masked=2, node_sizes=(20, 2))
    theta = I.make_params(wl, jitter=0.1)
    x, y = I.make_batch(wl)
    rng = np.random.default_rng(d + shared)
    tokens = x[:20].reshape(-1)
    tokens[:] = rng.integers(0, 200, tokens.size)
    tokens[rng.permutation(tokens.size)[:shared]] = 207
    x[:20] = tokens.reshape(x[:20].shape)
    x[20:] = np.arange(x[20:].size).reshape(x[20:].shape)
    x[20, 3] = 207
    gpu = run_gpu(wl, theta, x, y, flags=FUSED | NO_GRAPH)
    ref = oracle_steps(wl, theta, x, y)
    check_against_oracle(wl, gpu, ref)
    row, ref_row = gpu["G"][207 * d:208 * d], np.asarray(ref["G"])[207 * d:208 * d]
    assert np.linalg.norm(row - ref_row) <= TOL[wl.dtype] * np.linalg.norm(ref_row)


def test_encoder_fused_and_staged_agree_bitwise():
    wl, theta, x, y = _case("enc_small_bf16")
    a = run_gpu(wl, theta, x, y, flags=0)
    b = run_gpu(wl, theta, x, y, flags=FUSED)
    assert a["G"].tobytes() == b["G"].tobytes()


OVERLAP = 4


@pytest.mark.parametrize("name,sizes", [("enc_small_bf16", None), ("enc_small_bf16", [2, 2, 1, 3, 1]),
                                        ("enc_mid_bf16", [1, 1, 1, 1, 1]), ("enc_wide_bf16", None)])
def test_encoder_two_streams_agree_bitwise(name, sizes):
    """Forward passes on one stream, backward passes on the other (two sets of what passes from a
    node's forward to its backward part), staged and fused, replayed and launched one by one,
    three steps: the same bits as one stream."""
    print(f"case {name} sizes={sizes}", flush=True)
    wl, theta, x, y = _case(name)
    if sizes is not None:
        assert sum(sizes) == wl.batch
    base = run_gpu(wl, theta, x, y, node_sizes=sizes, flags=FUSED | NO_GRAPH, steps=3)
    assert base["streams"] == 1
    for flags in (OVERLAP, OVERLAP | NO_GRAPH, FUSED | OVERLAP, FUSED | OVERLAP | NO_GRAPH):
        other = run_gpu(wl, theta, x, y, node_sizes=sizes, flags=flags, steps=3)
        assert other["streams"] == 2, flags
        assert base["G"].tobytes() == other["G"].tobytes(), flags
        assert base["theta"].tobytes() == other["theta"].tobytes(), flags
        assert base["loss"] == other["loss"], flags
        assert base["node_losses"].tobytes() == other["node_losses"].tobytes(), flags


def test_encoder_fp32_keeps_one_stream():
    """The fp32 attention path shares its score scratch between the two passes: no second stream."""
    wl, theta, x, y = _case("enc_small_f32")
    assert run_gpu(wl, theta, x, y, flags=FUSED | OVERLAP | NO_GRAPH)["streams"] == 1


def test_encoder_two_steps():
    wl, theta, x, y = _case("enc_small_f32")
    gpu = run_gpu(wl, theta, x, y, steps=2)
    ref = oracle_steps(wl, theta, x, y, steps=2)
    check_against_oracle(wl, gpu, ref, tol=5e-4)


def test_encoder_partition_invariance_on_device():
    wl, theta, x, y = _case("enc_small_f32")
    a = run_gpu(wl, theta, x, y, node_sizes=[wl.batch])
    b = run_gpu(wl, theta, x, y, node_sizes=[1] * wl.batch)
    assert np.linalg.norm(b["G"] - a["G"]) <= 2e-5 * np.linalg.norm(a["G"])


def test_c4_full_size():
    """4-layer encoder 768/12/3072, T=128, vocab 30522, B=256 in 16 nodes of 16, Adam."""
    print("full size C4", flush=True)
    wl, theta, x, y = _case("C4", jitter=0.0)
    ref = oracle_steps(wl, theta, x, y)
    for flags, group in ((0, 0), (FUSED | OVERLAP | NO_GRAPH, 8)):      # the second is what bench.py times (the encoder takes 4 of the 8)
        print(f"flags {flags} group {group}", flush=True)
        gpu = run_gpu(wl, theta, x, y, flags=flags, node_group=group)
        check_against_oracle(wl, gpu, ref)
        check_update_from_own_gradient(wl, gpu, theta, tol=1e-4)
    # the bound that does not depend on where operands are rounded
    check_independent_bound(wl, gpu["G"], ref["G"], weights_only_gradient(wl, theta, x, y), "C4")


@pytest.mark.parametrize("group", [2, 4])
@pytest.mark.parametrize("name,sizes", [("enc_small_bf16", [2, 2, 2, 1, 1, 1]), ("enc_small_f32", [1] * 9),
                                        ("enc_mid_bf16", [1, 1, 1, 1, 1])])
def test_encoder_node_groups_match_the_oracle(name, sizes, group):
    """Groups of up to four consecutive nodes, of one size or of several, as one unit of the passes (the sequences of an encoder node are
    independent: only the loss bookkeeping tells the nodes apart): per-node losses and the combined
    gradient against the oracle, one and two streams bitwise equal."""
    wl, theta, x, y = _case(name)
    assert sum(sizes) == wl.batch
    ref = oracle_steps(wl, theta, x, y, node_sizes=sizes)
    base = None
    for flags in (FUSED, FUSED | NO_GRAPH, FUSED | OVERLAP | NO_GRAPH, 0):
        gpu = run_gpu(wl, theta, x, y, node_sizes=sizes, flags=flags, node_group=group)
        check_against_oracle(wl, gpu, ref)
        if base is None:
            base = gpu
        assert gpu["G"].tobytes() == base["G"].tobytes(), flags
        assert gpu["node_losses"].tobytes() == base["node_losses"].tobytes(), flags
