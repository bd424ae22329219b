// Fully connected ReLU network of the learned initial guess (FP32 on the
// device): forward, mean-squared-error gradients, Adam, and the scatter of
// its outputs into a right-hand-side-shaped solution vector.
#pragma once

#include <cstdint>
#include <string>
#include <vector>

namespace mlfma {

class Mlp;

Mlp* mlp_create(const std::vector<int>& sizes, uint64_t seed, std::string& err);
void mlp_destroy(Mlp* m);
int64_t mlp_num_params(const Mlp* m);
int mlp_get_params(const Mlp* m, float* host, std::string& err);
int mlp_set_params(Mlp* m, const float* host, std::string& err);
int mlp_inputs(const Mlp* m);
int mlp_outputs(const Mlp* m);
// Y [n][out] = net(X [n][in]), device pointers.
int mlp_forward(Mlp* m, const float* X, int n, float* Y, void* stream, std::string& err);
// loss = 0.5 / n * sum |net(X) - T|^2; grads (host, parameter layout) if not null.
int mlp_loss_grad(Mlp* m, const float* X, const float* T, int n, double* loss, float* grads, void* stream,
                  std::string& err);
// one Adam step; *loss = the loss before the step
int mlp_train_step(Mlp* m, const float* X, const float* T, int n, float lr, double* loss, void* stream,
                   std::string& err);
// The array and incidences of a learned guess.  Device tables of the particles
// (guess_tables_fill), host directions [R][3] and class parameters [C].
struct GuessInput {
  const int *cls = nullptr, *box_of = nullptr, *part_of_box = nullptr;
  const double *centers = nullptr, *khat = nullptr, *class_param = nullptr;
  double scale = 1, k = 0;
  int P = 0, C = 0, nx = 0, ny = 0, edge_cap = 0;
};
// x[r][p][j] = (Y[r*P+p][2j] + i Y[r*P+p][2j+1]) exp(-j k khat_r . c_p) in the
// context precision (0: complex float, 1: complex double), Y the network's
// outputs on the features of mlfma_guess_features (formed on the device).
int mlp_guess(Mlp* m, const GuessInput& in, int R, int n, int precision, void* x_dev, void* stream, std::string& err);

// The particle tables of one array on the device: copied on first use (and
// again if the current device changed), freed with the object.
struct GuessTables;
GuessTables* guess_tables_create();
void guess_tables_destroy(GuessTables* t);
int guess_tables_fill(GuessTables* t, const std::vector<int>& cls, const std::vector<int>& box_of,
                      const std::vector<int>& part_of_box, const std::vector<double>& centers, GuessInput& in,
                      std::string& err);

}  // namespace mlfma
