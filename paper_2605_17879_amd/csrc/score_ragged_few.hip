// The scoring kernel for rank counts that fill no tiling exactly: up to 8 192 ranks.
#define GD_SCORE_RAGGED 1
#include "score.hip"
