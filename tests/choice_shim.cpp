// Host entry points over the library's own choice of configuration and split,
// built by the CPU tests: the functions the calls use, not a copy of them.
#include "../paper_1904_05347_amd/csrc/pk_api.hip"

#include <new>

// Allocations of this library's own code, refused on demand.
static bool refuse_new = false;
void *operator new(size_t n)
{
    if (refuse_new) throw std::bad_alloc();
    return malloc(n);
}
void operator delete(void *p) noexcept { free(p); }
void operator delete(void *p, size_t) noexcept { free(p); }

extern "C" {

// The status of a look-up by name while allocations are refused; -1: an exception.
int shim_force_without_memory(const char *name)
{
    refuse_new = true;
    int st = -1;
    try {
        st = pk_force_config(name);
    } catch (...) {
    }
    refuse_new = false;
    pk_force_config(nullptr);
    return st;
}

// A configuration and its split: tile, K-block, groups of waves, stream-K,
// split, predicted time (us, -1 outside the model).
struct shim_pick {
    int64_t bm, bn, bk, kg, streamk, splits;
    double us;
};

static shim_pick describe(const pk::CostFamily &f, const Config *c, int64_t M, int64_t N, int64_t K, int splits)
{
    const int t = cost_tile(f, c);
    return {c->bm, c->bn, c->bk, c->kgroups, c->streamk, splits, t < 0 ? -1.0 : pk::predict_us(f, f.tiles[t], M, N, K, splits)};
}

static int held(int splits, int64_t M, int64_t N, size_t ws_bytes)
{
    return splits > 1 && ws_bytes < (size_t)splits * M * N * sizeof(float) ? 1 : splits;
}

int shim_wino_form(int m, int64_t T, int64_t Cin, int64_t Cout) { return pk::wino_form(m, T, Cin, Cout); }
int shim_wino_fused_fits(int m, int form, int64_t T, int64_t Cout) { return pk::wino_fused_fits(m, form, T, Cout); }

// The rule's configuration and the chosen one, each with its split as far as
// ws_bytes of workspace hold the partial sums.
void shim_gemm(int ta, int tb, int64_t M, int64_t N, int64_t K, int vec, size_t ws_bytes, shim_pick *rule, shim_pick *pick)
{
    const pk::CostFamily &f = vec ? pk::kCostGemm44 : pk::kCostGemm11;
    const int64_t lda = ta ? M : K, ldb = tb ? K : N;
    const Config *r = select_gemm_rule(ta, tb, M, N, K, lda, ldb, N, vec);
    *rule = describe(f, r, M, N, K, held(rule_gemm_splits(r, ta, tb, M, N, K, vec), M, N, ws_bytes));
    int s = 0;
    const Config *c = select_gemm(ta, tb, M, N, K, lda, ldb, N, vec, ws_bytes, &s);
    *pick = describe(f, c, M, N, K, held(s, M, N, ws_bytes));
}

// ... of a convolution (M outputs, K taps times channels; whole4: channels are
// multiples of four, as for va4 and vb4); a stream-K form without room for its
// plan gives way as it does in the call.
void shim_conv(int64_t M, int64_t Cout, int64_t K, int va4, int vb4, int whole4, size_t ws_bytes, shim_pick *rule, shim_pick *pick)
{
    const pk::CostFamily &f = va4 && vb4 ? pk::kCostConv44 : va4 ? pk::kCostConv41 : pk::kCostConv11;
    SkPlan plan;
    auto room = [&](const Config *c) { return !c->streamk || (streamk_plan(c, M, Cout, K, &plan) && ws_bytes >= plan.bytes); };
    const Config *r = select_conv_rule(M, Cout, K, va4, vb4, true, true);
    if (!room(r)) r = select_conv_rule(M, Cout, K, va4, vb4, true, false);
    *rule = describe(f, r, M, Cout, K, r->streamk ? 1 : held(choose_splits(r, M, Cout, K), M, Cout, ws_bytes));
    int s = 0;
    const Config *c = select_conv(M, Cout, K, va4, vb4, whole4, true, true, ws_bytes, &s);
    if (!room(c)) c = select_conv(M, Cout, K, va4, vb4, whole4, true, false, ws_bytes, &s);
    *pick = describe(f, c, M, Cout, K, held(s, M, Cout, ws_bytes));
}

// Records a measured configuration and split, as the automated search does.
int shim_record(int kind, int64_t M, int64_t N, int64_t K, int window, int stride, const char *config, int splits)
{
    return record_tuned({kind, 0, 0, M, N, K, window, stride, find_config(config)->name, splits});
}

}  // extern "C"
