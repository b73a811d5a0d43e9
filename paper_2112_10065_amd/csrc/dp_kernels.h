// Internal interface between the C-ABI layer (dp_api.hip) and the kernel files.
// Host-side launch functions take plain structs; no validation happens here.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

typedef unsigned short bf16_t;  // raw bfloat16 bits

enum : unsigned {
    KF_BIAS = 1u,     // add bias in the epilogue
    KF_RELU = 2u,     // max(.,0) in the epilogue
    KF_OUT_F32 = 4u,  // final output stored as fp32 instead of bf16
    KF_DB = 16u,      // backward-filter: also sum the bias gradient (kernels that cannot leave db_done unset)
    KF_MASK_IN = 8u,  // backward-data: dx *= [x > 0], x = the layer's saved input (output of the preceding ReLU)
    KF_NT_A = 32u,    // forward / backward-data: every weight is read by one block only (a single pixel tile): non-temporal loads, the stream leaves the caches alone
    KF_NT_OUT = 64u,  // backward-filter: a large gradient written once: non-temporal stores
    KF_FUSED_REDUCE = 256u,  // forward / backward-data with a reduction split: the block that finishes a tile last adds the splits' partial sums itself
};

enum { PASS_FWD = 0, PASS_DGRAD = 1, PASS_WGRAD = 2 };

// bits of the planner's `restr` (0 - 2: auto_plan_list)
enum {
    RESTR_SAVED = 8,   // backward-data with a saved output to mask dy by: the generic kernel does that while it loads, the others need a pass
    RESTR_ORDER = 32,  // forward with DP_RELU and without DP_RELU_IN: the default choice leaves out the kernel that adds in another order (forward_flat_plan)
    RESTR_BASE = 16,   // the kernels and prices that need least scratch: no flat-walk kernel in backward-data
    RESTR_WINDOW = 64,   // filter gradient: the window kernel in the place of the nine-tap one, whose blocks ask for more scratch
    RESTR_PATCH = 128,   // filter gradient, with RESTR_BASE: blocks and price of the nine-tap kernel as with the 256-pixel tiles of the wave-per-tap one
};

// Geometry of one conv layer plus its implicit-GEMM view for one pass.
//   fwd   : A rows = c_out,  B rows = output pixels (n,p,q), reduction = (r,s,c)
//   dgrad : A rows = c_in,   B rows = input pixels  (n,h,w), reduction = (r,s,k)
//   wgrad : A rows = c_out,  B rows = filter taps   (r,s,c), reduction = output pixels
// "A" / "B" are the matrix-core operands; D[i][j] has i over A rows, j over B rows.
struct ConvGeom {
    int N, H, W, C, K, R, S, sh, sw, ph, pw, Ho, Wo;
};

struct GemmPlan {
    int variant;          // tile variant index (see tile table in conv_mfma.hip)
    int TA, TB, BK;       // tile extents
    int tilesA, tilesB;   // tile counts
    int steps_total;      // reduction steps of BK
    int steps_per_split;  // steps handled by one split
    int splits;           // grid.y
    bool vecA, vecB;      // 16-byte loads allowed for operand A / B
    bool fast;            // fast-path kernel (conv_fast.hip) instead of the generic one
    bool dma;             // pipelined direct-to-LDS kernel (conv_dma.hip)
    bool halo = false;    // input-patch kernel (conv_halo.hip); implies dma
    int blocks = 0;       // persistent kernels: blocks per row tile (0: one per CU)
    bool phase = false;   // strided backward-data walks the input pixels stride phase by stride phase (conv_dma.hip)
    bool fill = false;    // phase, 1x1 filter: only the first phase has tiles, they store the zeros of the others
    bool wstrip = false;  // filter gradient with the x strip shared by the taps of a filter row (conv_wstrip.hip); implies dma
    bool win = false;     // forward / backward-data with one window of pixels for all taps (conv_win.hip); implies dma
    bool pw = false;      // 1x1 forward / backward-data with stationary weights (conv_pw.hip); implies dma
    bool pw_gather = false;  // pw, forward: strided or padded
    bool wwin = false;    // filter gradient with one window of x for all taps of a block (conv_wwin.hip); implies dma
    bool row_taps = false;   // wwin: three taps of one filter row per wave
    bool db_wave = false; // input-patch filter gradient: one more wave per block can sum the bias gradient (at most 15 taps)
    bool over_generic = false;   // a flat-walk kernel on a layer that the generic kernel would run otherwise
    bool fused_reduce = false;   // pipelined forward / backward-data with splits > 1: no second kernel, the last block of a tile reduces (conv_dma.hip)
};

struct ConvArgs {
    ConvGeom g;
    GemmPlan plan;
    int pass;
    unsigned flags;
    const bf16_t *x;      // fwd: x       dgrad: saved input for KF_MASK_IN, else -        wgrad: x
    const bf16_t *w;      // fwd: w       dgrad: w        wgrad: -
    const bf16_t *dy;     // fwd: -       dgrad: dy       wgrad: dy
    const bf16_t *ymask;  // saved post-ReLU output or nullptr (dgrad, wgrad)
    const float *bias;    // fwd
    void *out;            // fwd: y, dgrad: dx (bf16 or fp32), wgrad: dw (fp32)
    float *partial;       // [splits][rowsB][rowsA] (fwd/dgrad) or [splits][rowsA][rowsB] (wgrad)
    float *db_out = nullptr;      // KF_DB: bias gradient [rowsA]
    float *db_partial = nullptr;  // KF_DB: [splits][rowsA] scratch for split plans
    int db_rows = 0;              // > 0: db_partial holds this many rows of column sums from an earlier pointwise pass; the
                                  // split-reduce kernel adds them up into db_out (the main kernel does not touch them)
};

// dp_api.hip: timing hook of dp_trace_begin / dp_trace_end.  The launch function of every kernel family calls this right
// after it has enqueued the main kernel of a pass (before any split-reduce or column-sum kernel that follows).
void dp_trace_main_kernel_done(hipStream_t st);

// conv_wstrip.hip
hipError_t wstrip_init();
bool wstrip_plan(const ConvGeom &g, int force_splits, GemmPlan *pl);
hipError_t wstrip_launch(const ConvArgs &a, hipStream_t st);

// conv_win.hip
hipError_t win_init();
bool win_plan(const ConvGeom &g, int pass, int variant, GemmPlan *pl);
void win_kernel_name(int pass, const GemmPlan &pl, bool saved, char *name, size_t name_bytes);
hipError_t win_launch(const ConvArgs &a, hipStream_t st);
bool win_work(const ConvGeom &g, int pass, int variant, int *rounds, int *rows);   // channel rounds of a block, window rows copied in each

// conv_pw.hip
hipError_t pw_init();
bool pw_plan(const ConvGeom &g, int pass, int variant, int force_splits, GemmPlan *pl);
void pw_kernel_name(int pass, const GemmPlan &pl, bool masked, char *name, size_t name_bytes);   // masked: with the fused input-ReLU mask
int pw_blocks(const GemmPlan &pl);   // persistent blocks per channel tile
hipError_t pw_launch(const ConvArgs &a, hipStream_t st);

// conv_wwin.hip
hipError_t wwin_init();
bool wwin_plan(const ConvGeom &g, int slots_per_chunk, int force_splits, GemmPlan *pl);
void wwin_kernel_name(const GemmPlan &pl, char *name, size_t name_bytes);
hipError_t wwin_launch(const ConvArgs &a, hipStream_t st);

// conv_mfma.hip
hipError_t mfma_init();                                      // raises dynamic LDS limits
void mfma_plan(const ConvGeom &g, int pass, int force_variant, int force_splits, GemmPlan *plan);
size_t mfma_partial_bytes(const ConvGeom &g, int pass, const GemmPlan &plan);
hipError_t mfma_launch(const ConvArgs &a, hipStream_t st);
void mfma_kernel_name(int pass, const GemmPlan &plan, char *name, size_t name_bytes);
// sums a.partial into a.out; with_db: also a.db_partial [splits][rowsA] into a.db_out (backward-filter)
hipError_t launch_split_reduce(const ConvArgs &a, int rowsA, int rowsB, hipStream_t st, bool with_db = false);

// conv_fast.hip : fast path for channel counts that are multiples of the reduction step
hipError_t fast_init();
bool fast_plan(const ConvGeom &g, int pass, int force_variant, int force_splits, GemmPlan *plan);
hipError_t fast_launch(const ConvArgs &a, hipStream_t st);
void fast_kernel_name(int pass, const GemmPlan &plan, char *name, size_t name_bytes);

// true if this backward-filter plan's kernel sums the bias gradient itself when KF_DB is set
bool plan_sums_bias_gradient(const GemmPlan &plan);

// conv_dma.hip : multi-stage direct-to-LDS pipeline (forward, c_in % 64 == 0)
hipError_t dma_init();
bool dma_plan(const ConvGeom &g, int pass, int force_variant, int force_splits, GemmPlan *plan, bool f32_out = false);   // f32_out: fp32 input gradient
hipError_t dma_launch(const ConvArgs &a, hipStream_t st);
void dma_kernel_name(int pass, const GemmPlan &plan, char *name, size_t name_bytes);

// conv_halo.hip : input patch with halo resident in LDS (stride 1, 64 reduction channels per tap; 3x3 also 128)
hipError_t halo_init();
bool halo_plan(const ConvGeom &g, int pass, int force_variant, int force_splits, GemmPlan *plan);
hipError_t halo_launch(const ConvArgs &a, hipStream_t st);
bool dma_plan_is_flat(const GemmPlan &plan);    // the kernels that walk the reduction flat over (tap, channel)
int dma_plan_groups(const GemmPlan &plan);      // reduction groups of a block (1: the kernel has none)
bool dma_plan_is_strip(const GemmPlan &plan);   // the pixel-strip forward / backward-data kernels (no fused split reduction)
bool dma_fused_reduce_fits(int rowsA, int rowsB, int splits);
bool dma_plan_fuses_reduce(const GemmPlan &plan);   // the splits are summed by the main kernel: no reduction kernel follows
void halo_kernel_name(int pass, const GemmPlan &plan, bool masked, char *name, size_t name_bytes);   // masked: backward-data with the fused input-ReLU mask

// conv_fp32.hip : fp32 matrix instructions (reference-precision path)
hipError_t f32_conv_fwd(const ConvGeom &g, unsigned flags, const float *x, const float *w,
                        const float *bias, float *y, hipStream_t st);
hipError_t f32_conv_dgrad(const ConvGeom &g, const float *dy, const float *ymask, const float *w, const float *xin,
                          float *dx, hipStream_t st);   // xin (may be NULL): dx *= [xin > 0]
hipError_t f32_conv_wgrad(const ConvGeom &g, const float *x, const float *dy, const float *ymask,
                          float *dw, float *dbias, hipStream_t st);   // dbias may be NULL
void f32_kernel_name(const ConvGeom &g, int pass, bool masked, char *name, size_t name_bytes);   // as a profiler prints it; masked: a saved output masks dy

// pointwise.hip : ReLU-gradient / bias-gradient
size_t rbg_workspace_bytes(long long rows, int k);
hipError_t rbg_launch(long long rows, int k, bool bf16, const void *dy, const void *ymask,
                      void *g_out, float *dbias, float *ws, hipStream_t st);
// the first kernel only: column sums of `*row_blocks` row ranges in ws [row_blocks][k]; with one row block the sums
// go straight to dbias and nothing is left to add
hipError_t rbg_launch_partial(long long rows, int k, bool bf16, const void *dy, const void *ymask,
                              void *g_out, float *dbias, float *ws, hipStream_t st, int *row_blocks);
// sums ws [row_blocks][k] into dbias in row-block order
hipError_t rbg_launch_final(int k, int row_blocks, const float *ws, float *dbias, hipStream_t st);

// planner.hip : picks the cheapest fast-path variant and split for a pass (host-side cost model)
bool auto_plan(const ConvGeom &g, int pass, int force_splits, GemmPlan *plan, int restr = 0, double *time = nullptr);
// forward: the flat-walk plan that adds in the same order as `base` and is faster, if there is one
bool forward_flat_plan(const ConvGeom &g, const GemmPlan &base, GemmPlan *plan, double *time);
// backward-data: a flat-walk plan faster than `base`, whose price is `time`
bool backward_flat_plan(const ConvGeom &g, const GemmPlan &base, double time, int restr, GemmPlan *plan, double *flat_time);
// forward / backward-data: the window kernel's two cheapest plans, and whether it takes the place of `base`, whose price is `time`
bool pixel_window_exists(const ConvGeom &g, int pass);   // some tile of the window kernel runs the layer
int pixel_window_plans(const ConvGeom &g, int pass, GemmPlan out[2], double times[2], bool saved = false);
bool pixel_window_plan(const ConvGeom &g, int pass, const GemmPlan &base, double time, bool saved, double mask_us, GemmPlan *out);
// 1x1 layers by the kernel with stationary weights: its two cheapest plans, and whether it takes the place of `base` (masked: with the fused input-ReLU mask)
int pointwise_plans(const ConvGeom &g, int pass, bool masked, GemmPlan out[2], double times[2]);
bool pointwise_plan(const ConvGeom &g, int pass, const GemmPlan &base, bool masked, GemmPlan *out);
// filter gradient: the window kernel's two cheapest plans, and whether it takes the place of `base`, whose price is `time`
int wgrad_window_plans(const ConvGeom &g, GemmPlan out[2], double times[2]);
bool wgrad_window_plan(const ConvGeom &g, const GemmPlan &base, double time, GemmPlan *out);
bool wgrad_window_form(const ConvGeom &g, GemmPlan *out);
// the cheapest plans by the model, best first (input of the measured choice); returns the count
// restr: bit 0: fp32 gradients (not from kernels that stage bf16), bit 1: masked by the saved input, bit 2: the caller measures with cold caches; others above
int auto_plan_list(const ConvGeom &g, int pass, int force_splits, GemmPlan *out, int max_out, int restr = 0, double *times = nullptr);

// small_c.hip : explicit im2col for layers with very few input channels (c_in % 8 != 0, R*S*C <= 256)
int small_c_kpad(const ConvGeom &g);   // padded reduction length, 0 if the layer does not qualify
hipError_t small_c_im2col(const ConvGeom &g, int kpad, const bf16_t *x, bf16_t *xcol, hipStream_t st);
hipError_t small_c_pad_weights(const ConvGeom &g, int kpad, const bf16_t *w, bf16_t *wpad, hipStream_t st);
hipError_t small_c_unpad_dw(const ConvGeom &g, int kpad, const float *dwpad, float *dw, hipStream_t st);
// direct kernels without the im2col matrix (R*S*C <= 32, c_out % 8 == 0)
// dense_stream.hip: 1x1 layers over a few pixel rows (dense layers at small batch), one launch per pass that streams the weights
bool dense_fwd_stream_shape(const ConvGeom &g);
hipError_t dense_fwd_stream(const ConvGeom &g, unsigned flags, const bf16_t *x, const bf16_t *w, const float *bias, bf16_t *y, hipStream_t st);
bool dense_wgrad_stream_shape(const ConvGeom &g);
const char *dense_fwd_stream_name(const ConvGeom &g);     // kernel names as a profiler prints them
const char *dense_wgrad_stream_name(const ConvGeom &g);
hipError_t dense_wgrad_stream(const ConvGeom &g, const bf16_t *x, const bf16_t *dy, float *dw, float *db, hipStream_t st);
bool dense_dgrad_stream_shape(const ConvGeom &g);
hipError_t dense_dgrad_stream(const ConvGeom &g, unsigned flags, const bf16_t *dy, const bf16_t *w, const bf16_t *xin, void *dx, hipStream_t st);
// forward and backward-data in one pass over the weights (with_y false: backward-data alone, then y is NULL in the second call); the
// second call adds the partials and applies the epilogues
bool dense_both_shape(const ConvGeom &g);
bool dense_dgrad_split_shape(const ConvGeom &g);   // backward-data alone takes it
size_t dense_both_partial_bytes(const ConvGeom &g, bool with_y);
const char *dense_both_name(const ConvGeom &g, bool with_y);
hipError_t dense_both(const ConvGeom &g, const bf16_t *x, const bf16_t *dy, const bf16_t *w, float *partial, bool with_y, hipStream_t st);
hipError_t dense_both_sum(const ConvGeom &g, unsigned flags_y, unsigned flags_dx, const float *partial, const float *bias, const bf16_t *xin, bf16_t *y,
                          void *dx, hipStream_t st);
bool small_c_direct(const ConvGeom &g);
hipError_t small_c_fwd_direct(const ConvGeom &g, unsigned flags, const bf16_t *x, const bf16_t *w, const float *bias, bf16_t *y,
                              hipStream_t st);
// strided stems (7x7 stride 2 on RGB): forward straight from the input patch, no im2col matrix
bool small_c_stem(const ConvGeom &g);
hipError_t small_c_fwd_stem(const ConvGeom &g, unsigned flags, const bf16_t *x, const bf16_t *w, const float *bias, bf16_t *y, hipStream_t st);
// their filter gradient, unmasked dy, one fp32 partial per block; db (may be NULL) receives the bias gradient
bool small_c_wgrad_stem_shape(const ConvGeom &g);
int small_c_wgrad_stem_blocks(const ConvGeom &g);
size_t small_c_wgrad_stem_partial_bytes(const ConvGeom &g);
void small_c_wgrad_stem_name(const ConvGeom &g, char *name, size_t name_bytes);
hipError_t small_c_wgrad_stem(const ConvGeom &g, const bf16_t *x, const bf16_t *dy, float *partial, float *dw, float *db, hipStream_t st);
int small_c_wgrad_blocks(const ConvGeom &g, bool masked);   // pixel-range blocks, each writes one fp32 partial (masked: a saved output is applied to dy)
const char *small_c_wgrad_kernel(const ConvGeom &g, bool masked, bool with_db);   // name of the kernel that runs, as a profiler prints it
const char *small_c_fwd_kernel(const ConvGeom &g);
size_t small_c_wgrad_partial_bytes(const ConvGeom &g);
// ymask (saved output, may be NULL) masks dy on the fly; db (may be NULL) receives the bias gradient of the masked dy
hipError_t small_c_wgrad_direct(const ConvGeom &g, const bf16_t *x, const bf16_t *dy, const bf16_t *ymask, float *partial, float *dw,
                                float *db, hipStream_t st);
