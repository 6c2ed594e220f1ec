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
