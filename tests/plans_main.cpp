// The launch plans of the library, answered on the host: a line "gemm M N K", "accept B V", "logits B k V" or "attention B k Hq Hkv D P Lmax" or "lengths ..." in, the
// plan's numbers out.  Host code only; nothing here launches, so the few runtime calls that the sources make have empty bodies.
#ifdef PLANS_RUNTIME
extern "C" {
void* __hipRegisterFatBinary(void*) { return nullptr; }
void __hipRegisterFunction() {}
void __hipRegisterVar() {}
void __hipUnregisterFatBinary() {}
}
#else
#include "skinny_gemm.hip"
#include "spec_accept.hip"
#include "spec_accept_logits.hip"
#include "verify_attention.hip"
#include <cstdio>
#include <cstring>

int main() {
    char kind[16];
    while (scanf("%15s", kind) == 1) {
        if (!strcmp(kind, "gemm")) {
            int M, N, K;
            if (scanf("%d %d %d", &M, &N, &K) != 3) return 1;
            const lotts::GemmPlan p = lotts::plan_gemm(M, N, K);
            static const char* const forms[] = {"stream256", "stream128", "stream64", "direct"};
            printf("form %s rn %d tt %d nby %d ksplit %d\n", forms[p.form], p.rn, p.tt, p.nby, p.ksplit);
        } else if (!strcmp(kind, "accept")) {
            int B, V;
            if (scanf("%d %d", &B, &V) != 2) return 1;
            const lotts::FusedPlan p = lotts::plan_fused(B, V);
            printf("groups %d subs %d parts %d\n", p.iters, p.nsub, p.parts);
        } else if (!strcmp(kind, "logits")) {
            int B, k, V;
            if (scanf("%d %d %d", &B, &k, &V) != 3) return 1;
            const lotts::LgLayout l = lotts::lg_layout(B, k, V);
            printf("loads %d pieces %d\n", l.iters, l.npieces);
        } else if (!strcmp(kind, "attention")) {
            lotts_attn_desc d = {};
            d.dtype = LOTTS_BF16;
            if (scanf("%d %d %d %d %d %d %d", &d.B, &d.k, &d.Hq, &d.Hkv, &d.D, &d.P, &d.Lmax) != 7) return 1;
            const lotts::AttnPlan p = lotts::plan_attention(d);
            printf("one %d nqt %d fold %d shares %d prefix_shares %d merge %d\n", p.one, p.nqt, p.fold, p.nsplit_priv, p.nsplit_pre, p.merge);
        } else if (!strcmp(kind, "lengths")) {
            lotts_attn_desc d = {};
            d.dtype = LOTTS_BF16;
            if (scanf("%d %d %d %d %d %d %d", &d.B, &d.k, &d.Hq, &d.Hkv, &d.D, &d.P, &d.Lmax) != 7) return 1;
            const lotts::AttnPlans p = lotts::plan_attention(d);
            printf("flat %d workers %d merge %d nqt %d fold %d bytes %zu least %zu\n", p.flat, p.workers, p.flat ? p.flat_merge : p.merge, p.nqt, p.fold,
                   lotts::workspace_layout(d, p, nullptr, nullptr), lotts::workspace_layout(d, lotts::plan_attention(d, false), nullptr, nullptr));
        } else {
            return 1;
        }
    }
    return 0;
}
#endif
