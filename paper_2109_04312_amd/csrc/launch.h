// Host-side launchers, one per kernel family.  Everything is enqueued on `stream`.
#pragma once
#include <hip/hip_runtime.h>

#include <atomic>

#include "seg_layout.h"

namespace mate {

// Do the rows that an attention launch stores, `bytes_each` for an element of Q, pass through the L2 (see ResultRows)?  Where it is small there is nothing to overlap, and the launch waits for
// memory instead of the L2.  us, left and through: dense forward of 4 x 60, 12 heads (0.4 MB) 4.34 and 4.55, 4 x 128 (0.8 MB) 5.46
// and 5.65, 8 x 128 (1.6 MB) 5.57 and 5.67, 16 x 128 (3.1 MB) 5.86 and 5.80, 24 x 128 (4.7 MB) 7.50 and 7.17; segments, 12 heads, one
// sequence of 512 with its tables 14.93 and 14.98, 3 x 512 (2.4 MB) 8.27 and 8.22, 2 x 1000 10.03 and 9.78, 8 x 512 (6.3 MB) 11.27 and
// 10.69; f32, 6 x 106 with 4 heads and its tables 11.77 and 11.9, 4 x 512 (6.3 MB) 13.81 and 13.66; dense backward of 1 x 64, 4 heads (0.1
// MB) 5.79 and 5.95, 4 x 60, 12 heads (1.1 MB) 6.01 and 6.10, 4 x 128 (2.4 MB) 8.02 and 8.06, 8 x 128 (4.7 MB) 8.31 and 8.14.  The other
// backward kernels and the products pass it at any size: backward by segments, 12 heads, of 1 x 128 10.31 and 10.27, 1 x 512 14.60 and
// 14.31, 8 x 512 23.4 and 22.5, 1 x 2048 18.9 and 17.7, f32 of 1 x 128, 4 heads 11.66 and 11.77, 1 x 512, 12 heads 25.3 and 24.8; 768 wide, QKV
// at 64 tokens 7.22 and 7.21, 512 8.22 and 7.96, 8 x 512 19.3 and 17.6, output 7.10 and 7.10, 7.55 and 7.52, 10.7 and 10.1, both gradients of QKV at
// 300 16.4 and 15.8 (dW alone has a rule of its own).  (Zeros of pad rows always do: their workgroups end long before the launch.)
inline bool result_through(int B, int H, int N, int bytes_each) { return (size_t)B * H * N * 64 * bytes_each > (2u << 20); }

struct AttnArgs {
  const void *q, *k, *v;    // [B,H,N,64]
  const void *o, *dout;     // backward only
  void *out;                // forward only
  float* lse;               // forward: written; backward: read (const in spirit)
  void *dq, *dk, *dv;       // backward only
  float* delta;             // backward scratch [B,H,N]: rowsum(dO * O), negated in the bf16 path
  float* nlse;              // backward scratch [B,H,N] of the bf16 path: -lse / scale
  float* part[3];           // partial results of chunked question-token owners, per (b,h):
                            //   forward: [0] unnormalised O;  backward: dQ, dK, dV
  float* part_ml;           // forward: running max (log2 domain) and sum per partial row
  unsigned long long* arrived;     // one word per partial slot: which chunks have left their partials
  unsigned long long ticket;       // forward: what a chunk sets its word to, new for every call
  SegTables seg;
  alignas(4) unsigned char head_order[256];  // heads sorted column heads first (stable);
                                             // read as 32-bit words by the kernels
  int n_col;                      // number of column heads
  int B, H, N;
  float scale;
};

// Arguments of the dense-mask variant (no segment tables: ids and flags directly).
constexpr int kDenseMaxN = 1024;
struct DenseArgs {
  const void *q, *k, *v, *o, *dout;
  void* out;
  float* lse;
  void *dq, *dk, *dv;
  float *delta, *nlse;      // backward scratch [B,H,N]: -rowsum(dO * O), -lse / scale
  const int *row_ids, *col_ids;
  const unsigned char* flags;
  unsigned col_heads[8];    // one bit per head: words, because a byte would be fetched with a vector load
  int B, H, N;
  float scale;
};

// Measurement hook: when `kernel` matches the kernel about to be launched (or `also`, for a launch that does the
// work of two), record `start` before and `stop` after that one launch on its stream, then disarm.
struct ProfileHook {
  int kernel;
  hipEvent_t start, stop;
};
extern thread_local ProfileHook g_profile_hook;
struct ProfileScope {
  hipStream_t stream;
  bool armed;
  ProfileScope(int kernel, hipStream_t s, int also = -1)
      : stream(s), armed(g_profile_hook.kernel == kernel || g_profile_hook.kernel == also) {
    if (armed) (void)hipEventRecord(g_profile_hook.start, stream);
  }
  ~ProfileScope() {
    if (armed) {
      (void)hipEventRecord(g_profile_hook.stop, stream);
      g_profile_hook.kernel = 0;
    }
  }
};

// More than 64 KB of dynamic LDS has to be allowed explicitly, once per kernel and device (a host-side
// setting; the call costs a microsecond).
template <auto kKernel>
hipError_t allow_lds(int bytes) {
  static std::atomic<unsigned long long> done{0};  // bit = device
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  const unsigned long long bit = dev < 64 ? 1ull << dev : 0;
  if (bit && (done.load(std::memory_order_acquire) & bit)) return hipSuccess;
  e = hipFuncSetAttribute(reinterpret_cast<const void*>(kKernel), hipFuncAttributeMaxDynamicSharedMemorySize, bytes);
  if (e == hipSuccess) done.fetch_or(bit, std::memory_order_release);
  return e;
}

// max_global >= N and radius = 0: the pattern of Section 3; otherwise the bucketed approximation
// of Section 3.1 (global part of at most max_global tokens, windows of three buckets of radius).
hipError_t launch_build_segments(const int* row_ids, const int* col_ids,
                                 const unsigned char* flags, int B, int N, int max_global,
                                 int radius, int* seg, hipStream_t stream);

// Positional index restarting at each cell (Section 3.2); out is [B, N] int32.
hipError_t launch_cell_positions(const int* row_ids, const int* col_ids, const unsigned char* flags,
                                 int B, int N, int* out, hipStream_t stream);

// Projections either side of the attention (bf16): x [B,N,E] -> q, k, v [B,H,N,64] with
// w_qkv [3*H*64, E]; o [B,H,N,64] -> y [B,N,E] with w_o [E, H*64].  bias may be null.
// H even, E a multiple of 128.
hipError_t launch_qkv_project(const void* x, const void* w_qkv, const float* bias,
                              const unsigned char* flags, int B, int N, int H, int E, void* q,
                              void* k, void* v, hipStream_t stream);
hipError_t launch_out_project(const void* o, const void* w_o, const float* bias,
                              const unsigned char* flags, int B, int N, int H, int E, void* y,
                              hipStream_t stream);

// Backward of the two projections.  dx / d_o, dw, dbias may each be null (not wanted); dw and
// dbias are float32.  `workspace` holds *_project_bwd_workspace(...) bytes; `ticket`: see arrival.h.
size_t qkv_project_bwd_workspace(int B, int N, int H, int E);
size_t out_project_bwd_workspace(int B, int N, int H, int E);
hipError_t launch_qkv_project_bwd(const void* x, const void* w_qkv, const unsigned char* flags,
                                  const void* dq, const void* dk, const void* dv, int B, int N, int H,
                                  int E, void* dx, float* dw, float* dbias, void* workspace,
                                  unsigned long long ticket, hipStream_t stream);
hipError_t launch_out_project_bwd(const void* o, const void* w_o, const unsigned char* flags,
                                  const void* dy, int B, int N, int H, int E, void* d_o, float* dw,
                                  float* dbias, void* workspace, unsigned long long ticket, hipStream_t stream);

// Measurement aid: `workgroups` x 4 wavefronts each issue `iters` x 8 independent 32x32x16 bf16
// MFMAs and write one float per thread to `sink` (workgroups * 256 floats).
hipError_t launch_mfma_probe(float* sink, int workgroups, int iters, hipStream_t stream);
double mfma_probe_flop(int workgroups, int iters);

// fp32 matrix-core kernels: the path for dtype f32.
hipError_t launch_fwd_f32(const AttnArgs& a, hipStream_t stream);
hipError_t launch_bwd_f32(const AttnArgs& a, hipStream_t stream);

// bf16 MFMA kernels.
hipError_t launch_fwd_mfma(const AttnArgs& a, hipStream_t stream);
hipError_t launch_bwd_mfma(const AttnArgs& a, hipStream_t stream);
hipError_t launch_fwd_dense(const DenseArgs& a, hipStream_t stream);
hipError_t launch_bwd_dense(const DenseArgs& a, hipStream_t stream);

}  // namespace mate
