// The form that the proxy's GEMM takes: lines of "M N K" in, lines of "name,blocks,threads of a block" out.
#include <cstdio>

#include "../../paper_2406_10707_amd/csrc/gemm_forms.hpp"

int main() {
    int m, n, k;
    while (scanf("%d %d %d", &m, &n, &k) == 3) {
        const dsllm::GemmForm &f = dsllm::kGemmForms[dsllm::gemm_form(m, n, k)];
        printf("%s,%llu,%d\n", f.name, (unsigned long long)f.tiles_m(m) * f.tiles_n(n), f.threads);
    }
}
