// Plans of several updates per unroll, without a GPU: the library's host code on handles that only have a configuration.
// argv: seed and number of shapes.  Prints "ok <shapes>" or the first shape that is wrong.
#include <stdio.h>
#include <unistd.h>
#include <random>
#include "../../paper_2104_06272_amd/csrc/anakin.hip"

struct Shape { anakin_env_cfg env; anakin_net_cfg net; int B, T, n; };

static Shape shape(int kind, int rows, int cols, std::initializer_list<int> hidden, int dtype, int B, int T, int n)
{
    Shape s;
    memset(&s, 0, sizeof s);
    s.env.kind = kind; s.env.rows = rows; s.env.cols = cols; s.env.max_steps = 9;
    s.net.policy = kind == ANAKIN_ENV_PENDULUM ? ANAKIN_POLICY_TANH_GAUSSIAN : ANAKIN_POLICY_CATEGORICAL;
    for (int w : hidden) s.net.hidden[s.net.n_hidden++] = w;
    s.net.dtype = dtype; s.net.gamma = 0.99f; s.net.lambda_ = 1.0f; s.net.lr = 1e-3f; s.net.beta1 = 0.9f; s.net.beta2 = 0.999f; s.net.eps = 1e-8f;
    s.B = B; s.T = T; s.n = n;
    return s;
}

// false: the library does not take the shape at all
static bool check(const Shape& s)
{
    anakin h{};
    std::string err;
    if (build_shapes(&s.env, &s.net, s.B, s.T, h.env, h.net, err) != ANAKIN_OK) return false;
    h.env_cfg = s.env; h.net_cfg = s.net; h.B = s.B; h.T = s.T; h.n_updates = 1;
    plan(h.env, h.net, s.B, s.T, h.splits, h.quanta, &h.splits_w, &h.head_fan, &h.loss_blocks);
    if (h.loss_blocks < s.B / 8) h.loss_blocks = s.B / 8;
    auto bad = [&](const char* what) {
        printf("%s: env %d (%d x %d) hidden", what, s.env.kind, s.env.rows, s.env.cols);
        for (int l = 0; l < s.net.n_hidden; ++l) printf(" %d", s.net.hidden[l]);
        printf(" dtype %d B %d T %d updates %d: %s\n", s.net.dtype, s.B, s.T, s.n, h.err.c_str());
        fflush(stdout); _exit(1);
    };
    const int rc = anakin_set_updates_per_unroll(&h, s.n);
    if (s.T % s.n) { if (rc != ANAKIN_E_BAD_CONFIG) bad("accepted although T is no multiple"); return true; }
    if (rc != ANAKIN_OK) bad("refused");
    if (h.n_updates != s.n) bad("number of updates not set");
    if (s.n == 1) return true;
    // every region's partial sums fit the room of the full unroll, and no workgroup starts behind the last sample
    const int M = s.B * (s.T / s.n), L = h.net.L;
    for (int l = 0; l <= L; ++l) {
        if (h.sub_splits[l] < 1 || h.sub_splits[l] > h.splits[l]) bad("chunks");
        if ((long long)(h.sub_splits[l] - 1) * chunk_rows(M, h.sub_splits[l], h.sub_quanta[l]) >= M) bad("empty chunk");
    }
    const int stage = h.sub_splits[L] * h.sub_head_fan;
    if (h.sub_head_fan < 1 || (h.sub_head_fan > 1 && (h.head_fan < 2 || stage > h.splits[L] * h.head_fan))) bad("first stage of the head gradient");
    if ((long long)(stage - 1) * chunk_rows(M, stage, h.sub_quanta[L]) >= M) bad("empty workgroup of the head gradient");
    if ((h.sub_splits_w > 0) != (h.splits_w > 0) || h.sub_splits_w > h.splits_w) bad("wall plane");
    if (h.sub_loss_blocks * s.n > h.loss_blocks + s.T) bad("loss partials");
    return true;
}

int main(int argc, char** argv)
{
    std::mt19937 rng(argc > 1 ? atoi(argv[1]) : 1);
    const int want = argc > 2 ? atoi(argv[2]) : 1000;
    auto pick = [&](std::initializer_list<int> v) { return v.begin()[rng() % v.size()]; };
    int done = 0;
    // one-layer nets whose head gradient takes the two-level sum, in chunks that would fan out further than the full unroll
    done += check(shape(ANAKIN_ENV_CATCH, 10, 5, {256}, ANAKIN_DTYPE_FP32, 3200, 32, 4));
    done += check(shape(ANAKIN_ENV_CATCH, 10, 5, {32}, ANAKIN_DTYPE_BF16, 3200, 32, 4));
    done += check(shape(ANAKIN_ENV_PENDULUM, 0, 0, {128}, ANAKIN_DTYPE_BF16, 7808, 64, 4));
    if (done != 3) { printf("a fixed shape is not taken\n"); fflush(stdout); _exit(1); }
    while (done < want) {
        const int kind = pick({ANAKIN_ENV_CATCH, ANAKIN_ENV_PENDULUM, ANAKIN_ENV_MAZE}), T = 1 + rng() % 64;
        Shape s = shape(kind, 2 + rng() % 15, 2 + rng() % 15, {}, pick({ANAKIN_DTYPE_FP32, ANAKIN_DTYPE_BF16}), pick({16, 64, 256}) * (1 + rng() % (1 << rng() % 9)), T, 1 + rng() % T);
        if (rng() % 4) s.n = pick({1, 2, 2, 4, 8}), s.T = s.n * (1 + T / s.n);
        s.net.n_hidden = 1 + rng() % 3;
        for (int l = 0; l < s.net.n_hidden; ++l) s.net.hidden[l] = pick({32, 64, 128, 256, 512});
        done += check(s);
    }
    printf("ok %d\n", done);
    fflush(stdout);
    _exit(0);                                                    // no GPU: nothing of the runtime to take down
}
