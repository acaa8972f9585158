// The top-k passes without the workgroups that are there for the guesses (BPC_TOPK_FIRST_GUESS), as if
// something else on the device kept them from running: workgroups that have waited leave every partition to the
// long form.  Built by __graft_entry__.build(), used by test_gpu_late_guess.py.
#define BPC_TOPK_FIRST_GUESS 0
#define bpc bpc_late
#include "../paper_2105_07829_amd/csrc/cluster.hip"
#include "../paper_2105_07829_amd/csrc/dense.hip"
#include "../paper_2105_07829_amd/csrc/topk.hip"

extern "C" {
// As bpc_compress and bpc_server_aggregate, of top-k alone, without their checks.
int late_compress(const bpc_params_t *prm, const void *grad, int dtype, float *residual, uint64_t D, void *payload, void *ws,
                  void *stream) {
  bpc::Source src{};
  src.grad = grad;
  src.dtype = dtype;
  src.residual = residual;
  return (int)bpc::topk_encode(bpc::make_geo(prm, D), *prm, nullptr, src, (uint8_t *)payload,
                               bpc::Workspace{(uint8_t *)ws, bpc::ws_layout(prm, D)}, (hipStream_t)stream);
}
int late_aggregate(const bpc_params_t *prm, const void *const *payloads, int n, float *residual, uint64_t D, void *payload, void *ws,
                   void *stream) {
  bpc::Source src{};
  src.residual = residual;
  src.msgs.n = n;
  src.msgs.inv_n = 1.0f / (float)n;
  for (int i = 0; i < n; ++i) src.msgs.ptr[i] = (const uint8_t *)payloads[i];
  return (int)bpc::topk_encode(bpc::make_geo(prm, D), *prm, nullptr, src, (uint8_t *)payload,
                               bpc::Workspace{(uint8_t *)ws, bpc::ws_layout(prm, D)}, (hipStream_t)stream);
}
}
