// Shape support, chunk limits and workspace sizing of the matrix-core path.
#include "m2rnn_kernels.hpp"
#include "m2rnn_mfma_common.hpp"

namespace m2rnn {

int mfma_bwd_max_chunk(int K, int V);

bool mfma_supported(int K, int V) { return mfma_pick_rb(K, V, 1 << 20) != 0; }

// The chunk is bounded by the backward's on-chip stash; the default is the
// largest that fits (fewest checkpoint bytes).
int mfma_max_chunk(int K, int V) { return mfma_bwd_max_chunk(K, V); }
int mfma_default_chunk(int K, int V) { return mfma_bwd_max_chunk(K, V); }

namespace {
size_t part_bytes(int B, int T, int N, int V) { return (size_t)B * T * N * V * 4; }
}  // namespace

size_t mfma_fwd_least_bytes(int B, int T, int N, int K, int V) {
  const int rb = mfma_pick_rb(K, V, B * N);
  const int P = rb ? K / (16 * rb) : 1;
  return P > 1 ? align256(P * part_bytes(B, T, N, V)) : 0;
}

size_t mfma_fwd_workspace_bytes(int B, int T, int N, int K, int V) {
  const size_t least = mfma_fwd_least_bytes(B, T, N, K, V);
  if (!half_serves(K, V, B * N, T)) return least;
  const int P = K / (8 * half_pick_rb(K, V, B * N, 0, 0, T));
  const size_t want = P > 1 ? align256(P * part_bytes(B, T, N, V)) : 0;
  return want > least ? want : least;
}

}  // namespace m2rnn
