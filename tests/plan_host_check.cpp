// Host-side check of the launch plans (tests/test_batch_plans.py): for every
// minibatch size that hieravg_set_batch takes, what its plan reads and writes
// must fit the buffers that create sizes.  Built from the library's host code
// alone; plans need no GPU.
#include <cstdio>
#include <random>

#include "hieravg.hip"

namespace {

struct Handle {
  hieravg* h = new hieravg;
  ~Handle() { delete h; }
};

// A handle as hieravg_create_config has it before its buffers exist.
bool prepare(hieravg* h, const hieravg_config& c) {
  if (validate(c) != HIERAVG_OK) return false;
  h->cfg = c;
  h->T = c.k_global > 0 ? c.k_global : c.K1 * c.K2;
  h->cfg.k_global = h->T;
  h->cfg.K2 = (h->T + c.K1 - 1) / c.K1;
  set_dims(h);
  h->Bmax = c.B;
  return true;
}

int checked = 0, delayed_plans = 0, fails = 0;

void check(const hieravg_config& c) {
  Handle H;
  hieravg* h = H.h;
  if (!prepare(h, c)) return;
  const PlanNeed have = plan_need_upto(h, c.B);
  h->once_alloc = have.once;
  for (int B = 1; B <= c.B; ++B) {
    // as after a round of another minibatch size, delayed or from the common copy
    h->in_delayed = h->in_wg = true;
    const PlanNeed n = plan_need(h, B);
    if ((h->in_delayed && !n.delayed) || (h->in_wg && !n.once)) {
      ++fails;
      std::printf("FAIL B %d of %d keeps the schedule of the round before\n", B, c.B);
      return;
    }
    ++checked;
    delayed_plans += n.delayed ? 1 : 0;
    const bool ok = n.part <= have.part && n.part2 <= have.part2 && n.partv <= have.partv && n.gram <= have.gram &&
                    n.errors <= have.errors && (!n.delayed || have.delayed) && (!n.hb || have.hb) &&
                    (!n.once || have.once);
    if (!ok) {
      ++fails;
      std::printf("FAIL P %d S %d K1 %d K2 %d in %ld hidden %ld classes %ld B %d of %d: part %ld/%ld errors %ld/%ld "
                  "gram %ld/%ld delayed %d/%d\n", c.P, c.S, c.K1, c.K2, (long)c.in_dim, (long)c.hidden,
                  (long)c.classes, B, c.B, (long)n.part, (long)have.part, (long)n.errors, (long)have.errors,
                  (long)n.gram, (long)have.gram, n.delayed, have.delayed);
      return;
    }
  }
}

hieravg_config mlp(int P, int S, int K1, int K2, int B, long in, long hidden, long classes) {
  hieravg_config c{};
  c.P = P, c.S = S, c.K1 = K1, c.K2 = K2, c.B = B;
  c.kind = HIERAVG_KIND_MLP;
  c.in_dim = in, c.hidden = hidden, c.classes = classes, c.n_samples = 5000;
  c.noise_std = 0.5f, c.lr = 0.1f;
  return c;
}

}  // namespace

int main() {
  // Clusters whose rows pass K1 * S * B <= 16384 at a size whose padded form
  // does not: 113 .. 120, 81 .. 85, 97 .. 102, 33 .. 47 and (32 samples) 17 .. 27.
  check(mlp(17, 17, 8, 1, 128, 3072, 1024, 10));
  check(mlp(32, 32, 6, 2, 128, 3072, 512, 10));
  check(mlp(40, 20, 8, 1, 128, 3072, 1024, 100));
  check(mlp(43, 43, 8, 1, 48, 3072, 1024, 10));
  check(mlp(75, 75, 8, 1, 32, 256, 512, 10));
  std::mt19937 rng(1);
  auto pick = [&](int lo, int hi) { return (int)(lo + rng() % (unsigned)(hi - lo + 1)); };
  for (int i = 0; i < 3000; ++i) {
    const int S = 1 << pick(0, 7), K1 = pick(1, 8);
    hieravg_config c = mlp(0, S + pick(0, S - 1), K1, pick(1, 3), pick(1, 200), pick(1, 5000), pick(1, 1100),
                           i % 3 ? pick(2, 32) : pick(33, 120));
    c.P = c.S * pick(1, 3);
    if (i % 4 == 0) c.momentum = 0.9f;
    if (i % 5 == 0) c.weight_decay = 1e-4f;
    if (i % 7 == 0) c.k_global = pick(1, 20);
    c.update_mode = i % 2 ? HIERAVG_UPDATE_AUTO : pick(0, 2);
    if (i % 6 == 0) c.kind = HIERAVG_KIND_SOFTMAX;
    check(c);
  }
  std::printf("%d plans, %d delayed\n", checked, delayed_plans);
  std::printf("%s\n", fails ? "plan checks FAILED" : "plan checks ok");
  return fails || delayed_plans < 1000;
}
