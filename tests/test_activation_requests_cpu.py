"""Which bytes the tiled prefill kernel's requests for activations touch, from the functions that the kernel itself uses: whatever a
lane's own offset lets through a resource lies inside the activations, and every column that is multiplied is brought to its place."""
import os
import subprocess

import pytest

import paper_2511_11248_amd as tman

CSRC = os.path.join(os.path.dirname(os.path.abspath(tman.__file__)), "csrc")

PROGRAM = r"""
#include <cstdio>
#include <cstdlib>
#include <vector>
#include "tman_activation_requests.h"
using namespace tman;
int main(int argc, char** argv) {
    const int K = atoi(argv[1]), tokens = atoi(argv[2]), rows_of_tile = 256, stages = K / 32;
    const uint32_t row = (uint32_t)K * 2u, bytes = (uint32_t)tokens * row;
    if (resource_bytes(bytes, (stages + 1) / 2, stages) != 0) return printf("a pair past K has a resource\n"), 1;
    for (int pair = 0; 2 * pair < stages; ++pair) {
        const uint32_t at = (uint32_t)pair * kPairBytes, size = resource_bytes(bytes, pair, stages);
        std::vector<int> seen(tokens * (kPairBytes / 16), 0);
        for (int q = 0; q < rows_of_tile / 8; ++q)
            for (int lane = 0; lane < 64; ++lane) {
                const uint32_t off = (uint32_t)(8 * q + (lane >> 3)) * row + request_chunk(q, lane);
                const int token = 8 * q + (lane >> 3), place = lane & 7, chunk = place ^ ((token >> 1) & 7);
                const bool read = off + 16 <= size;
                if (read && at + off + 16 > bytes) return printf("pair %d request %d lane %d leaves the activations\n", pair, q, lane), 1;
                const bool wanted = token < tokens && 64 * pair + 8 * chunk < K;
                if (wanted && (!read || at + off != token * row + (64 * pair + 8 * chunk) * 2u))
                    return printf("pair %d request %d lane %d: not chunk %d of token %d\n", pair, q, lane, chunk, token), 1;
                if (wanted) ++seen[token * 8 + chunk];
            }
        for (int t = 0; t < tokens; ++t)
            for (int c = 0; c < 8; ++c)
                if (seen[t * 8 + c] != (64 * pair + 8 * c < K)) return printf("pair %d token %d chunk %d: %d times\n", pair, t, c, seen[t * 8 + c]), 1;
    }
    return 0;
}
"""


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    folder = tmp_path_factory.mktemp("requests")
    source, binary = folder / "requests.cpp", folder / "requests"
    source.write_text(PROGRAM)
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Werror", "-I", CSRC, str(source), "-o", str(binary)], check=True)
    return str(binary)


@pytest.mark.parametrize("K", [32, 64, 96, 160, 544, 2656, 4096, 11008])
@pytest.mark.parametrize("tokens", [1, 33, 255, 256])
def test_requests_stay_inside_the_activations(program, K, tokens):
    r = subprocess.run([program, str(K), str(tokens)], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout


@pytest.mark.parametrize("K", [32, 96, 160, 2592])
@pytest.mark.parametrize("N", [1, 33, 300])
def test_what_follows_the_integer_activations_is_their_own(K, N):
    """The int8 kernels request 128 columns of a token at a time: up to 96 bytes behind the last token are still the buffer's."""
    assert tman.tman_act_i8_bytes(N, K) - N * K >= 96
