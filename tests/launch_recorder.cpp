// What libmpe asks of the HIP runtime, without a device: this program defines the runtime's functions that the library calls,
// so its own take their place (the executable comes first in symbol lookup), and prints every launch and every LDS
// attribute.  Memory is host memory, kernels do not run.  argv[1]: compute units (256).  Commands on stdin, one a line; after each one line "rc <n>":
//   create <scenario> <agents> <landmarks> <adversaries> <envs> <runs> [<hidden> <weight type> <steps of an episode> [<reward mode>]]
//                                                                        128 1 25 0
//   destroy | reset | set_state | gru | critic | mlp | mlp_critic | rollout <T> | rollout_ac <T> | abs_step
//   kernels                                                              the names of all that the library has
//   counters <unit>                                                      what mpe_set_state's kernel finds from here on (0)
//   fail <attribute|launch> <k>                                          the k-th such call from here on fails, once
#include <cxxabi.h>

#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <iostream>
#include <map>
#include <sstream>
#include <string>
#include <vector>

#include "../include/mpe.h"

namespace {
std::map<const void*, std::string>& kernels() {
  static std::map<const void*, std::string> m;
  return m;
}
struct Config { uint32_t grid[3], block[3]; size_t lds; void* stream; } pushed;
int last_error = 0;
int units = 256;           // compute units
uint32_t counters = 0;     // see the command
int fail_in[2] = {0, 0};   // attribute, launch: calls until the one that fails
int outcome(int kind) { return fail_in[kind] && --fail_in[kind] == 0 ? (last_error = 1) : 0; }
struct Dim3 { uint32_t x, y, z; };
}  // namespace

extern "C" {
void** __hipRegisterFatBinary(const void*) { static void* handle; return &handle; }
void __hipUnregisterFatBinary(void**) {}
void __hipRegisterVar(void**, void*, char*, char*, int, size_t, int, int) {}
void __hipRegisterFunction(void**, const void* host, char*, const char* name, unsigned, void*, void*, void*, void*, int*) {
  int status = 0;
  char* plain = abi::__cxa_demangle(name, nullptr, nullptr, &status);
  std::string s = status == 0 ? plain : name;
  std::free(plain);
  for (const char* drop : {"void ", "mpe::(anonymous namespace)::", "mpe::"})
    for (size_t at; (at = s.find(drop)) != std::string::npos;) s.erase(at, std::strlen(drop));
  kernels()[host] = s.substr(0, s.find('('));
}
int __hipPushCallConfiguration(Dim3 grid, Dim3 block, size_t lds, void* stream) {
  pushed = {{grid.x, grid.y, grid.z}, {block.x, block.y, block.z}, lds, stream};
  return 0;
}
int __hipPopCallConfiguration(Dim3* grid, Dim3* block, size_t* lds, void** stream) {
  *grid = {pushed.grid[0], pushed.grid[1], pushed.grid[2]};
  *block = {pushed.block[0], pushed.block[1], pushed.block[2]};
  *lds = pushed.lds;
  *stream = pushed.stream;
  return 0;
}
int hipLaunchKernel(const void* host, Dim3 grid, Dim3 block, void** args, size_t lds, void*) {
  const int rc = outcome(1);
  const std::string& name = kernels()[host];
  auto word = [&](int k) { return *static_cast<const uint32_t*>(args[k]); };
  std::printf("launch %s grid %u %u block %u lds %zu", name.c_str(), grid.x, grid.y, block.x, lds);
  if (name.rfind("rollout_gru_kernel<", 0) == 0) std::printf(" first %u groups %u", word(5), word(6));
  if (name.rfind("rollout_gru_waves_kernel<", 0) == 0) std::printf(" envs %u", word(4));
  if (name == "read_counters_kernel" && rc == 0) **static_cast<uint32_t**>(args[2]) = counters;
  std::printf("%s\n", rc ? " FAILS" : "");
  return rc;
}
int hipFuncSetAttribute(const void* host, int, int bytes) {
  const int rc = outcome(0);
  std::printf("attribute %s %d%s\n", kernels()[host].c_str(), bytes, rc ? " FAILS" : "");
  return rc;
}
int hipGetLastError() { const int e = last_error; last_error = 0; return e; }
const char* hipGetErrorString(int) { return "planned failure"; }
int hipGetDevice(int* dev) { *dev = 0; return 0; }
int hipDeviceGetAttribute(int* value, int, int) { *value = units; return 0; }
int hipDeviceSynchronize() { return 0; }
int hipMalloc(void** p, size_t n) { std::printf("malloc %zu\n", n); return (*p = std::calloc(n ? n : 1, 1)) ? 0 : 2; }
int hipFree(void* p) { std::free(p); return 0; }
int hipHostMalloc(void** p, size_t n, unsigned) { return (*p = std::calloc(n, 1)) ? 0 : 2; }
int hipHostFree(void* p) { std::free(p); return 0; }
int hipHostGetDevicePointer(void** dev, void* host, unsigned) { *dev = host; return 0; }
int hipMemcpyAsync(void*, const void*, size_t, int, void*) { return 0; }
int hipGetSymbolAddress(void** p, const void*) { *p = nullptr; return 1; }
}

int main(int argc, char** argv) {
  if (argc > 1) units = std::atoi(argv[1]);
  mpe_env* env = nullptr;
  alignas(16) static float w[4];                // never read: kernels do not run
  const float* p = w;
  std::string line;
  while (std::getline(std::cin, line)) {
    std::istringstream in(line);
    std::string what;
    in >> what;
    int rc = 0;
    if (what == "create") {
      mpe_config c{};
      in >> c.scenario >> c.num_agents >> c.num_landmarks >> c.num_adversaries >> c.num_envs >> c.num_runs;
      c.hidden = 128;
      c.weight_dtype = MPE_WEIGHTS_BF16;
      c.max_episode_steps = 25;
      if (int32_t hidden, dtype, steps; in >> hidden >> dtype >> steps) {
        c.hidden = hidden;
        c.weight_dtype = dtype;
        c.max_episode_steps = steps;
        if (in >> c.reward_mode) c.local_ratio = 0.5f;
      }
      c.dt = 0.1f; c.damping = 0.25f; c.mass = 1.0f; c.accel = 5.0f; c.agent_radius = 0.15f; c.landmark_radius = 0.05f;
      c.contact_force = 100.0f; c.contact_margin = 1e-3f;
      c.adv_radius = 0.075f; c.adv_accel = 3.0f; c.adv_max_speed = 1.0f; c.good_max_speed = 1.3f;
      rc = mpe_create(&c, &env);
    } else if (what == "destroy") {
      rc = mpe_destroy(env);
      env = nullptr;
    } else if (what == "reset") {
      rc = mpe_reset(env, 1u, nullptr, nullptr);
    } else if (what == "set_state") {
      rc = mpe_set_state(env, p, p, p, reinterpret_cast<const int32_t*>(p), 1u, 0u, nullptr);
    } else if (what == "gru") {
      rc = mpe_set_gru_policy(env, p, p, p, p, p, p, p, p, p, p, nullptr);
    } else if (what == "critic") {
      rc = mpe_set_gru_critic(env, p, p, p, p, nullptr);
    } else if (what == "mlp") {
      rc = mpe_set_policy(env, p, p, p, p, p, p, nullptr);
    } else if (what == "mlp_critic") {
      rc = mpe_set_critic(env, p, p, p, p, p, p, nullptr);
    } else if (what == "kernels") {
      for (const auto& k : kernels()) std::printf("kernel %s\n", k.second.c_str());
    } else if (what == "counters") {
      in >> counters;
    } else if (what == "rollout" || what == "rollout_ac") {
      int T = 0;
      in >> T;
      rc = what == "rollout" ? mpe_rollout(env, T, nullptr, nullptr, nullptr, nullptr, nullptr, nullptr)
                             : mpe_rollout_ac(env, T, nullptr, nullptr, nullptr, nullptr, nullptr, nullptr, nullptr, nullptr, nullptr);
    } else if (what == "abs_step") {
      uint32_t step = 0;
      rc = mpe_get_state(env, nullptr, nullptr, nullptr, nullptr, &step, nullptr);
      std::printf("abs_step %u\n", step);
    } else if (what == "fail") {
      std::string kind;
      int k = 0;
      in >> kind >> k;
      fail_in[kind == "launch"] = k;
    } else {
      return 2;
    }
    std::printf("rc %d\n", rc);
    std::fflush(stdout);
  }
  return 0;
}
