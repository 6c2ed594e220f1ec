"""The rules that choose the gate's kernel, on the host.  The points are those where one kernel measured clearly slower than the
one chosen (times at the rules in gate.hip)."""
import ctypes as C

import pytest

import paper_2205_10034_amd as M


def gate_kernel(T, d, E, packed, dtype="bf16", k=2):
    f = M.lib().moe_test_gate_kernel
    f.restype, f.argtypes = C.c_char_p, [C.c_void_p, C.c_int32]
    c = M.MoEConfig(T=T, d_model=d, d_ff=64, E=E, k=min(k, E), dtype=dtype).c()
    return f(C.byref(c), packed).decode()


@pytest.mark.parametrize("E,d,T,want", [
    (64, 2048, 1024, "float64"), (64, 2048, 4096, "float64"), (64, 2048, 4097, "packed"), (64, 2048, 6000, "packed"),
    (64, 2048, 8191, "packed"), (64, 2048, 8192, "packed"), (64, 1024, 4096, "float64"), (64, 1024, 4097, "packed"),
    (64, 4096, 4096, "float64"), (64, 4096, 1024, "packed"), (64, 4096, 4097, "packed"), (64, 4096, 8191, "packed"),
    (40, 4096, 3072, "packed"), (48, 3072, 1024, "packed"), (63, 2048, 2048, "packed"), (33, 512, 4096, "float64"),
    (24, 2048, 1024, "split"), (24, 4096, 4096, "split"), (24, 2048, 4097, "packed"), (24, 2048, 6000, "packed"), (24, 1024, 4096, "float64"),
    (24, 512, 8191, "float64"), (24, 512, 16384, "packed"), (31, 2048, 3000, "float64"), (16, 2048, 8192, "split"), (8, 4096, 16384, "packed"),
    (64, 2048, 1000, "split"), (64, 2048, 16, "few"), (64, 2048, 17, "split")])
def test_gate_of_a_layer_with_a_packed_router(E, d, T, want):
    assert gate_kernel(T, d, E, 1) == want


@pytest.mark.parametrize("E,d,T,want", [
    (64, 2048, 4097, "float64"), (64, 4096, 4097, "split"), (48, 3072, 8193, "split"), (48, 3072, 6000, "float64"), (64, 4096, 8192, "float64"),
    (24, 1536, 6000, "float64"), (24, 2048, 1536, "split"), (24, 4096, 16384, "split"), (31, 4096, 4097, "float64"), (63, 4096, 4097, "float64"),
    (65, 64, 1, "float64"), (16, 2048, 4096, "split"), (17, 64, 1023, "split"), (17, 64, 1024, "float64")])
def test_gate_without_a_packed_router(E, d, T, want):
    assert gate_kernel(T, d, E, 0) == want


def test_float32_activations_always_take_the_exact_kernels():
    for E in (1, 7, 16, 64, 200):
        for T in (17, 1024, 9000):
            assert gate_kernel(T, 1024, E, 1, "f32") == gate_kernel(T, 1024, E, 0, "f32") == "float64"


def layer_routing(T, d, E, k, f=2048, alone=0, packed=0, dtype="bf16"):
    fn = M.lib().moe_test_layer_routing
    fn.restype, fn.argtypes = C.c_char_p, [C.c_void_p, C.c_int32, C.c_int32]
    c = M.MoEConfig(T=T, d_model=d, d_ff=f, E=E, k=k, dtype=dtype).c()
    return fn(C.byref(c), packed, alone).decode()


RANKED, RANK, SLICES, ONE = "parts + ranking product", "parts + ranking", "slices", "one token"


@pytest.mark.parametrize("T,d,E,k,want", [
    (2, 64, 4, 2, SLICES), (16, 2048, 64, 8, SLICES), (17, 2048, 65, 2, SLICES), (96, 1472, 9, 2, SLICES), (97, 1472, 9, 2, "split"),
    (97, 1536, 9, 2, SLICES), (256, 2048, 32, 4, SLICES), (257, 2048, 32, 3, "split"), (256, 2048, 33, 2, "split"),  # 8192 logits at most
    (32, 256, 256, 8, SLICES), (33, 256, 256, 8, "float64"), (128, 2048, 64, 8, SLICES), (129, 2048, 8, 8, "split"),  # 1024 assignments
    (1, 2048, 64, 1, SLICES), (1, 2048, 32, 1, ONE), (1, 2048, 24, 1, SLICES)])
def test_routing_of_a_layer(T, d, E, k, want):
    for packed in (0, 1):
        for alone in (0, 1):
            assert layer_routing(T, d, E, k, alone=alone, packed=packed) == want


def test_routing_of_a_layer_needs_room_for_the_partial_logits():
    # h has 128 bytes a token, a slice 8 E
    assert layer_routing(8, 2048, 16, 1, f=64) == SLICES and layer_routing(8, 2048, 17, 1, f=64) == "split"


@pytest.mark.parametrize("d,E,k,f,layer,alone", [
    (2048, 64, 2, 8192, RANKED, RANK), (4096, 33, 8, 2048, RANKED, RANK), (2048, 65, 2, 8192, SLICES, SLICES), (1024, 24, 2, 2048, RANKED, RANK),
    (64, 64, 2, 64, ONE, ONE), (64, 33, 2, 64, "split", "split"), (64, 33, 2, 128, RANK, RANK), (128, 33, 2, 64, "split", "split")])
    # (the last four: no room for a slice in yd and h, in yd, in h)
def test_routing_of_a_one_token_layer(d, E, k, f, layer, alone):
    assert layer_routing(1, d, E, k, f) == layer and layer_routing(1, d, E, k, f, alone=1) == alone


def test_routing_of_a_float32_layer_is_the_gate():
    for T in (1, 8, 256):
        assert layer_routing(T, 2048, 33, 2, dtype="f32") == "float64"
