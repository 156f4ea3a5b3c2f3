// Coarse-grid MLP (device state and host driver); see mlp.hip.
#pragma once
#include <vector>

#include "hhg_internal.h"

namespace hhg {

// Offsets and (padded) shapes of the four weight matrices in the parameter vector.
struct WShapes {
  long off[4];
  int rows[4], cols[4];
};

struct AdamArgs;
struct PackArgs;

struct Mlp {
  int n_in = 0, hidden = 0, n_out = 0, max_batch = 0;
  int kin = 0, kout = 0, bpad = 0;     // padded to multiples of 16
  int rows[4], cols[4];                // device layer shapes (padded)
  long woff[4], boff[4], nparams_dev = 0;
  float *P = nullptr, *Gr = nullptr, *Mo = nullptr, *Vo = nullptr;  // params, grads, Adam moments (float32)
  unsigned short* Pb = nullptr;        // bf16 copy of the params
  unsigned short* PbT = nullptr;       // bf16 transposed weight matrices (same offsets, cols x rows)
  unsigned short* A0[2] = {nullptr, nullptr};   // bf16 input (this minibatch and the next)
  unsigned short* A0T[2] = {nullptr, nullptr};  // and transposed (kin x bpad), for the weight gradients
  float* Zout = nullptr;               // output of a forward call, padded (float32)
  unsigned short* Ab[3] = {nullptr, nullptr, nullptr};            // bf16 hidden activations
  unsigned short* AbT[3] = {nullptr, nullptr, nullptr};           // transposed (rows x bpad)
  unsigned short* G[4] = {nullptr, nullptr, nullptr, nullptr};    // bf16 gradients wrt pre-activations
  unsigned short* GT[4] = {nullptr, nullptr, nullptr, nullptr};   // transposed (rows x bpad)
  double* partial = nullptr;
  double* loss_acc = nullptr;          // device loss accumulator (2 doubles)
  long step = 0;
  std::vector<void*> allocs;

  ~Mlp();
  void init(int n_in, int hidden, int n_out, int max_batch);
  long host_params() const;                       // unpadded parameter count
  void set_params(const float* host);             // host order W1,b1,...,W4,b4 (row-major W)
  void unpack(const float* dev_vec, float* host) const;
  void transpose_weights(hipStream_t s);           // PbT from Pb
  WShapes shapes() const;
  void forward(hipStream_t s, const float* x, int B, float* y);
  PackArgs pack_args(const float* x, const int* idx, int B, bool train, int buf) const;
  void forward_layers(hipStream_t s, int B, int buf, const float* y, const int* idx);
  // adds the batch's mean loss to loss_acc[0] on the device (no host sync)
  void loss_grad_dev(hipStream_t s, const float* y, const int* idx, int B, int buf, double* loss_acc,
                     const AdamArgs& adam, const PackArgs& next);
  double loss_grad(hipStream_t s, const float* x, const float* y, int B);  // grads in Gr
  // Adam steps of every full minibatch of every epoch: order (device) holds
  // n_samples rows of the data sets x, y per epoch; loss[e] += the batch losses
  void train_dev(hipStream_t s, const float* x, const float* y, int n_samples, int batch, int epochs, float lr,
                 const int* order, double* loss);
};

}  // namespace hhg
