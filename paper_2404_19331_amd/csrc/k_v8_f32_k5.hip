#define FCM_DT TF32
#define FCM_DT_NAME "f32"
#define FCM_K 5
#define FCM_KNAME "5"
#define FCM_TABLE_FN variants_v8_f32_k5
#define FCM_V8_TABLE FCM_V8(2, 0, 1), FCM_V8(2, 2, 1), FCM_V8(4, 0, 1), FCM_V8(4, 4, 1)
#include "k_v8.inc"
