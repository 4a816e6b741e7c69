// Build-time generator of the register-resident couplings.
//
// BisContract<L, B, R> (bisector, Appendix F coefficients in the real-harmonic basis):
//   run(a, w, E)      E_l += sum_nu w_{l nu} sum S Re(conj(a_p1) a_p2)   (one k mode)
//   targets(a, T)     T_{l nu} = sum S Re(conj(a_p1) a_p2)               (one k mode)
//   run_orders(a, w, E)  E_{beta, l} += sum_nu w_{l nu} sum S^beta Re(conj(a_p1) a_p2): the
//                     terms of each order theta^(2 beta) into an accumulator of their own
// MidReweight<L, K, ALLP, R> (midpoint; parity-even: Appendix D coefficients in the real basis,
//   all-parity: Section 3.2's phi with the sign (-1)^J2 of g folded in):
//   dirs(x, y, z, yD)   y_J1^mu1 of a unit vector at yD[J1*J1 + J1 + mu1], J1 <= K (parity-even: even J1)
//   parity_part(yD, y2, other)  yD <- the part of J1's parity (other: the other part) of a function that
//                       is yD at D and y2 at its mirror
//   chunk<C>(g, yD, Dp, A)  A_{l nu} += sum_{alpha>0} sum Phi' y_J1^mu1(D^) |D|^alpha g_{alpha J2 mu2} over
//   the g fields [kMixFields * C, kMixFields * (C + 1)) of the canonical order, g their values.
//   The canonical order is (alpha, J, mu): alpha = 2, 4, .., K with J even <= L + alpha, or every
//   alpha = 1 .. K with J = alpha mod 2, +2, .. <= L + alpha; Dp[alpha / 2] (all-parity: Dp[alpha])
//   is |D|^alpha and A runs over l = 2, 4, .., L; nu = -l .. l.  The monopole has no alpha > 0 term.
// Every coupling value comes from the host FP64 generator as a literal.
// Usage: gen_contract <contract_gen.inc> <mix_gen.inc>
#include <cmath>
#include <cstdio>
#include <map>
#include <utility>
#include <vector>

#include "coeffs.h"

namespace {

// g fields of the midpoint P_l in the canonical order
struct GField {
  int alpha, J, mu;
};
std::vector<GField> mid_fields(int L, int K, bool all) {
  std::vector<GField> v;
  for (int a = all ? 1 : 2; a <= K; a += all ? 1 : 2)
    for (int j = a % 2; j <= L + a; j += 2)
      for (int m = -j; m <= j; ++m) v.push_back(GField{a, j, m});
  return v;
}

int a_index(int l, int nu) {  // l = 2, 4, ...
  int p = 0;
  for (int ll = 2; ll < l; ll += 2) p += 2 * ll + 1;
  return p + nu + l;
}

// Straight-line evaluation of the real harmonics y_J^mu(x, y, z), J <= K (even J only unless
// `all`), by the Cartesian recurrences
//   Q_m^m = 1, Q_J^m = (2J-1)/(J-m) z Q_{J-1}^m - (J+m-1)/(J-m) Q_{J-2}^m,
//   y_J^{+-m} = norm_Jm Q_J^m(z) {Re, Im} (x + i y)^m.
void emit_dirs(FILE *f, int K, bool all) {
  std::fprintf(f, "  __device__ __forceinline__ static void dirs(R x, R y, R z, R *yD) {\n");
  std::fprintf(f, "    const R c0 = (R)1, s0 = (R)0;\n");
  for (int m = 1; m <= K; ++m)
    std::fprintf(f, "    const R c%d = c%d * x - s%d * y, s%d = c%d * y + s%d * x;\n", m, m - 1, m - 1, m, m - 1, m - 1);
  for (int m = 0; m <= K; ++m)
    for (int J = m; J <= K; ++J) {
      if (J == m) std::fprintf(f, "    const R q%d_%d = (R)1;\n", J, m);
      else if (J == m + 1) std::fprintf(f, "    const R q%d_%d = (R)%d * z;\n", J, m, 2 * m + 1);
      else
        std::fprintf(f, "    const R q%d_%d = (R)%.17g * z * q%d_%d - (R)%.17g * q%d_%d;\n", J, m,
                     (2.0 * J - 1) / (J - m), J - 1, m, (J + m - 1.0) / (J - m), J - 2, m);
      if (!all && (J & 1)) continue;
      double ratio = 1.0, dfm = 1.0;  // (J-m)!/(J+m)! and (2m-1)!!
      for (int i = J - m + 1; i <= J + m; ++i) ratio /= (double)i;
      for (int i = 2 * m - 1; i > 1; i -= 2) dfm *= (double)i;
      const double nrm = std::sqrt((2.0 * J + 1) / (4.0 * 3.14159265358979323846) * ratio) * dfm *
                         (m > 0 ? std::sqrt(2.0) : 1.0);
      if (m == 0) std::fprintf(f, "    yD[%d] = (R)%.17g * q%d_%d;\n", J * J + J, nrm, J, m);
      else
        std::fprintf(f, "    yD[%d] = ((R)%.17g * q%d_%d) * c%d; yD[%d] = ((R)%.17g * q%d_%d) * s%d;\n", J * J + J + m,
                     nrm, J, m, m, J * J + J - m, nrm, J, m, m);
    }
  std::fprintf(f, "  }\n");
  std::fprintf(f, "  __device__ __forceinline__ static void parity_part(R *yD, const R *y2, bool other) {\n"
                  "    const R e = other ? (R)-0.5 : (R)0.5;\n");
  if (all) std::fprintf(f, "    const R o = -e;\n");
  for (int J = 0; J <= K; J += all ? 1 : 2)
    for (int m = -J; m <= J; ++m)
      std::fprintf(f, "    yD[%d] = (R)0.5 * yD[%d] + %s * y2[%d];\n", J * J + J + m, J * J + J + m, (J & 1) ? "o" : "e",
                   J * J + J + m);
  std::fprintf(f, "  }\n");
}

// MidReweight<L, K, all>; false on an inconsistent field set.
bool emit_mid(FILE *f, int L, int K, bool all) {
  const std::vector<GField> fields = mid_fields(L, K, all);
  std::map<std::pair<int, std::pair<int, int>>, int> at;
  for (size_t i = 0; i < fields.size(); ++i) at[{fields[i].alpha, {fields[i].J, fields[i].mu}}] = (int)i;
  const int NG = (int)fields.size(), NCH = (NG + pw::kMixFields - 1) / pw::kMixFields;
  int NA = 0;
  for (int l = 2; l <= L; l += 2) NA += 2 * l + 1;
  std::fprintf(f, "template <typename R> struct MidReweight<%d, %d, %s, R> {\n", L, K, all ? "true" : "false");
  std::fprintf(f, "  static constexpr int NG = %d, NA = %d, NCH = %d;\n", NG, NA, NCH);
  emit_dirs(f, K, all);
  // chunk -> (Dp index, J1 mu1 index) -> local g index -> [(coef, A index)]: one weighted value at a
  // time is live, and every term is one multiply-add into its A
  typedef std::map<int, std::vector<std::pair<double, int>>> Users;
  std::vector<std::map<std::pair<int, int>, Users>> by((size_t)NCH);
  for (int alpha = all ? 1 : 2; alpha <= K; alpha += all ? 1 : 2)
    for (const pw::Term &t : all ? pw::midpoint_terms_all(L, alpha) : pw::midpoint_terms(L, alpha)) {
      if (t.l == 0) {
        // the monopole carries no line-of-sight dependence: its alpha > 0 couplings vanish
        if (t.c > 1e-12 || t.c < -1e-12) {
          std::fprintf(stderr, "gen_contract: non-zero monopole coupling at alpha=%d\n", alpha);
          return false;
        }
        continue;
      }
      auto it = at.find({alpha, {t.J2, t.mu2}});
      if (it == at.end()) {
        std::fprintf(stderr, "gen_contract: field (alpha=%d, J=%d, mu=%d) outside the field set\n", alpha, t.J2, t.mu2);
        return false;
      }
      const int p = it->second;
      by[(size_t)(p / pw::kMixFields)][{all ? alpha : alpha / 2, pw::sh_index(t.J1, t.mu1)}][p % pw::kMixFields]
          .push_back({t.c, a_index(t.l, t.nu)});
    }
  std::fprintf(f, "  template <int C> __device__ __forceinline__ static void chunk(const R *g, const R *yD, const R *Dp, R *A) {\n");
  for (int c = 0; c < NCH; ++c) {
    std::fprintf(f, "    if constexpr (C == %d) {\n", c);
    for (auto &grp : by[(size_t)c]) {
      std::fprintf(f, "      {\n        const R w = yD[%d] * Dp[%d];\n", grp.first.second, grp.first.first);
      for (auto &gi : grp.second) {
        std::fprintf(f, "        { const R h = w * g[%d];", gi.first);
        for (auto &ca : gi.second) std::fprintf(f, " A[%d] += (R)%.17g * h;", ca.second, ca.first);
        std::fprintf(f, " }\n");
      }
      std::fprintf(f, "      }\n");
    }
    std::fprintf(f, "    }\n");
  }
  std::fprintf(f, "  }\n};\n");
  return true;
}

}  // namespace

int main(int argc, char **argv) {
  if (argc < 3) {
    std::fprintf(stderr, "usage: gen_contract <contract.inc> <mix.inc>\n");
    return 2;
  }
  FILE *f = std::fopen(argv[1], "w");
  if (!f) return 1;
  std::fprintf(f, "// Generated by gen_contract.cpp at build time; do not edit.\n");
  // (L, K, all-parity) of the midpoint P_l
  const struct {
    int L, K;
    bool all;
  } mid_shapes[] = {{2, 2, false}, {2, 4, false}, {2, 6, false}, {4, 2, false}, {4, 4, false}, {4, 6, false},
                    {6, 2, false}, {6, 4, false}, {2, 1, true},  {2, 2, true},  {2, 3, true},  {2, 4, true},
                    {4, 1, true},  {4, 2, true},  {4, 3, true},  {4, 4, true}};
  const int lmaxs[] = {0, 2, 4, 6};
  for (int L : lmaxs)
    for (int B = 0; B <= 2; ++B) {
      const int J = L + B;
      const int NF = (J + 1) * (J + 1);
      std::vector<pw::Term> terms = pw::bisector_terms(L, B);
      std::map<std::pair<int, int>, std::vector<pw::Term>> by;
      for (const pw::Term &t : terms) by[{t.l, t.nu}].push_back(t);
      std::fprintf(f, "template <typename R> struct BisContract<%d, %d, R> {\n", L, B);
      std::fprintf(f, "  static constexpr bool kGenerated = true;\n");
      std::fprintf(f, "  static constexpr int NF = %d;\n", NF);
      std::fprintf(f, "  static constexpr int NTERMS = %d;\n", (int)terms.size());
      std::fprintf(f, "  static constexpr int NO = %d;\n", B + 1);
      for (int variant = 0; variant < 2; ++variant) {
        if (variant == 0)
          std::fprintf(f, "  __device__ __forceinline__ static void run(const cplx<R> *a, const R *w, R *E) {\n");
        else
          std::fprintf(f, "  __device__ __forceinline__ static void targets(const cplx<R> *a, R *T) {\n");
        for (auto &kv : by) {
          const int l = kv.first.first, nu = kv.first.second;
          std::fprintf(f, "    {\n      R t = (R)0;\n");
          for (const pw::Term &t : kv.second) {
            const int p1 = pw::sh_index(t.J1, t.mu1), p2 = pw::sh_index(t.J2, t.mu2);
            std::fprintf(f, "      t += (R)%.17g * (a[%d].x * a[%d].x + a[%d].y * a[%d].y);\n", t.c, p1,
                         p2, p1, p2);
          }
          if (variant == 0)
            std::fprintf(f, "      E[%d] += w[%d] * t;\n    }\n", l / 2, l * l + l + nu);
          else
            std::fprintf(f, "      T[%d] = t;\n    }\n", l * l + l + nu);
        }
        std::fprintf(f, "  }\n");
      }
      // one accumulator per order: E[beta * (L/2 + 1) + l/2]
      std::fprintf(f, "  __device__ __forceinline__ static void run_orders(const cplx<R> *a, const R *w, R *E) {\n");
      for (int beta = 0; beta <= B; ++beta) {
        std::map<std::pair<int, int>, std::vector<pw::Term>> byb;
        for (const pw::Term &t : pw::bisector_terms(L, beta, beta)) byb[{t.l, t.nu}].push_back(t);
        for (auto &kv : byb) {
          const int l = kv.first.first, nu = kv.first.second;
          std::fprintf(f, "    {\n      R t = (R)0;\n");
          for (const pw::Term &t : kv.second) {
            const int p1 = pw::sh_index(t.J1, t.mu1), p2 = pw::sh_index(t.J2, t.mu2);
            std::fprintf(f, "      t += (R)%.17g * (a[%d].x * a[%d].x + a[%d].y * a[%d].y);\n", t.c, p1,
                         p2, p1, p2);
          }
          std::fprintf(f, "      E[%d] += w[%d] * t;\n    }\n", beta * (L / 2 + 1) + l / 2, l * l + l + nu);
        }
      }
      std::fprintf(f, "  }\n");
      std::fprintf(f, "};\n");
    }
  std::fprintf(f, "struct MidShape { int L, K, all, NG; };\nconstexpr MidShape kMidShapes[] = {\n");
  for (const auto &sh : mid_shapes)
    std::fprintf(f, "  {%d, %d, %d, %d},\n", sh.L, sh.K, sh.all ? 1 : 0, (int)mid_fields(sh.L, sh.K, sh.all).size());
  std::fprintf(f, "};\n");
  std::fclose(f);
  f = std::fopen(argv[2], "w");
  if (!f) return 1;
  std::fprintf(f, "// Generated by gen_contract.cpp at build time; do not edit.\n");
  std::fprintf(f, "#define PW_MIX_SHAPES(X)");
  for (const auto &sh : mid_shapes) std::fprintf(f, " X(%d, %d, %s)", sh.L, sh.K, sh.all ? "true" : "false");
  std::fprintf(f, "\n");
  for (const auto &sh : mid_shapes)
    if (!emit_mid(f, sh.L, sh.K, sh.all)) return 1;
  std::fclose(f);
  return 0;
}
